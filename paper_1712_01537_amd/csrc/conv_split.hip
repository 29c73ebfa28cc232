// Stride-1 fp32 octree convolution on the bf16 matrix cores: every fp32
// operand is the sum of three bf16 parts (split3.h).
#include "conv_split.h"

#include <algorithm>

#include "pool_fuse.h"
#include "split3.h"

namespace {

typedef oc::s3_v4f v4f;
typedef oc::s3_v2u v2u;
typedef oc::s3_v4u v4u;

constexpr int TB = 512;
constexpr int WAVES = TB / 64;

// Rows of c channels at depth l too large for 32-bit byte offsets (BIG below).
bool rows_big(const oc_octree* t, int l, int c) {
  return t->N[l] * c * 4 >= int64_t(1) << 32;
}

// Raw buffer resource over `bytes` bytes at p: loads past its end return zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000);
}

// Two transposing LDS loads, the second `next` bytes behind the first: the eight
// rows (two times four) of this lane's channel.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
__device__ __forceinline__ v4u tr2(const char* p, int next) {
  const auto* a = (const __attribute__((address_space(3))) char*)p;
  const v2u lo = __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)a));
  const v2u hi =
      __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(a + next)));
  return v4u{lo[0], lo[1], hi[0], hi[1]};
}

// ---------------------------------------------------------------------------
// Stride-1, K = 3 convolution, weights in registers (k_conv_sp3):
// out[i][n] = sum_k sum_c x[nb(i,k)][c] W'[k][c][n] for the 16-channel chunk
// c0 = 16 blockIdx.z of the reduction (partial sums when there are several).
// The MFMA (16x16x32) computes out^T: A = W'^T (16 output channels x 32), B =
// the gathered rows (32 x 16 octants), where 32 = two taps x 16 channels: lane
// l supplies channels 8 (q & 1) .. + 7 of the pair's first (q < 2) or second
// tap, q = l / 16.  The 27 taps make 14 pairs: x-offsets 0 and 1 at each of
// the nine (y, z), then y-offsets 0 and 1 at x-offset 2, then the last three.
//
// A workgroup has eight waves: WN blocks of 16 output channels, WM = 4 / WN
// shares of the row blocks, and two halves of the tap pairs, whose sums meet
// through LDS.  A wave keeps the parts of its half's weights of its 16 output
// channels in registers for the whole launch (7 x 3 x 4 per lane), so the LDS
// holds x alone.  Workgroups (one per CU) are persistent over a contiguous
// range of sibling groups, taken in tiles of GPB groups (GPB/2 blocks of 16
// rows, RB per wave).
//
// One barrier per tile.  Between two of them tile t is multiplied, the rows of
// tile t+1, loaded a tile earlier, are split and stored to the other LDS
// buffer, those of tile t+2 are loaded, and the first half's waves add the
// second half's sums of tile t-1 to their own and write the result.  The first
// half does the multiplying last and the second half first: each SIMD has one
// wave of either, so one splits while the other multiplies.
//
// LDS layout, in 16-byte chunks (eight channels of one part of one position):
// part p, channel half h, group g, position (x, y, z) at
// (2p + h) HS + 72 g + 18 x + 4 y + z.  The strides 1, 4, 18 = 2 and 72 = 8
// (mod 16) put the 16 rows of a read (two groups' eight children) on distinct
// banks, and every tap is an immediate offset.  HS = 0 (mod 16): a 16-byte
// read serves lanes of two quarters of the wave in one cycle (0-3, 12-15 and
// 20-27; HS = 8 was measured to take twice the cycles).
//
// FLIP: input gradient, W'[k][c][n] = W[26-k][n][c].
// POOL (forward only, one reduction chunk): the 2x2x2 max-pool follows the
// (ReLU'd) output in the epilogue, through a small LDS area per wave; out is
// then the pooled map [npar][nn] of depth l-1 (row prow[g] for group g, loaded
// a tile ahead), psw the switches [ngroups][nn], and the workgroups of column
// block 0 zero an equal share of the rows of empty depth-(l-1) octants
// (plab[i] == 0).
// BIG: x is 4 GiB or more, too large for 32-bit offsets.
// Every lambda of the tile loop is inlined by force: one that is not, as the
// compiler decided for <4, 8, false, true, false>, takes wr, acc and prq by
// address and so puts them in scratch memory (16 -> 64 pooled, 69765 groups: 492
// us instead of 190).
//
// Measured on an MI355X (this kernel alone, forward; before: the fp32 MFMA
// kernel this one replaced, 16x16x4, weights in registers): 16->64 channels on
// 67121 groups of depth 6 145 us, 205 TFLOP/s of fp32 products (pooled 151);
// 32->64 on 4434 groups of depth 4 29 us (42); 16->16 on 211730 groups of depth
// 8 174 us (270).  At many groups and 64 channels the MFMAs run at 1.25 PFLOP/s
// of bf16; a plain bf16 matrix product reaches 1.24 at 8192 and 1.35 at 16384.
// With few groups per workgroup (about four tiles) the first loads and the
// weights' parts take 6 of 29 us; with 16 output channels the split and store
// of x (46 us of 61 at 67121 groups when the MFMAs were left out), which four
// waves' columns would share, bound it.
constexpr int NST = 14;  // tap pairs
struct Pair {
  int a, b;  // taps, b < 0: none
};
constexpr Pair pair_of(int s) {
  return s < 9 ? Pair{s, s + 9}
               : s < 12 ? Pair{18 + (s - 9), 21 + (s - 9)} : s == 12 ? Pair{24, 25} : Pair{26, -1};
}
constexpr int XS = 18, YS = 4, GS = 72;
constexpr int tap_off(int k) { return (k / 9) * XS + (k / 3 % 3) * YS + k % 3; }

// The barrier orders LDS accesses only: loads from global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int WN, int GPB, bool FLIP, bool POOL, bool BIG>
__global__ __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_sp3(
    const int32_t* __restrict__ nbr, int64_t ngroups, const float* __restrict__ x, int kk,
    const float* __restrict__ w, int nn, float* __restrict__ out, int relu,
    float* __restrict__ part, const int32_t* __restrict__ prow, const int32_t* __restrict__ plab,
    int64_t npar, uint8_t* __restrict__ psw) {
  constexpr int BN = 16 * WN, WM = WAVES / 2 / WN;
  constexpr int RB = GPB / 2 / WM;  // row blocks per wave
  static_assert(RB >= 1 && RB * WM * 2 == GPB, "every row block has two waves");
  constexpr int HS = GPB * GS, PS = 2 * HS, BUFC = 3 * PS;  // 16-byte chunks
  static_assert(HS % 16 == 0, "conflict-free reads");
  constexpr int NU = GPB * 256 / TB;  // (position, channel quad) units per thread
  __shared__ __attribute__((aligned(16))) v4u X[2 * BUFC];
  __shared__ __attribute__((aligned(16))) v4f EX[2][WAVES / 2][RB * 64];
  __shared__ __attribute__((aligned(16))) float PL[WAVES / 2][POOL ? oc::kPoolLdsFloats : 4];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, q = lane >> 4;
  const int th = wave >> 2, wv = wave & 3;  // tap half
  const int wn = wv % WN, wm = wv / WN;
  const int n0 = blockIdx.y * BN + 16 * wn, c0 = 16 * blockIdx.z;
  const int nx = gridDim.x, bx = blockIdx.x;
  const int lb = nx >= 8 ? (bx % 8) * (nx / 8) + bx / 8 : bx;  // XCD-contiguous ranges
  const int64_t g0 = ngroups * lb / nx, g1 = ngroups * (lb + 1) / nx;  // groups [g0, g1)
  const int T = (int)((g1 - g0 + GPB - 1) / GPB);
  if constexpr (POOL) {
    if (blockIdx.y == 0) {  // rows of empty depth-(l-1) octants
      const int64_t r0 = npar * lb / nx, r1 = npar * (lb + 1) / nx;
      const int c4 = nn / 4, cnt = (int)(r1 - r0) * c4;
      for (int e = tid; e < cnt; e += TB) {
        const int64_t i = r0 + e / c4;
        if (plab[i] == 0)
          *reinterpret_cast<v4f*>(out + i * nn + 4 * (e % c4)) = v4f{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  if (T <= 0) return;  // uniform over the workgroup

  const oc::SplitK sk = oc::s3_consts();
  // staging: thread -> channel quad, position, groups (tid >> 8) + 2 i
  const int f_ = tid & 3, pos = (tid >> 2) & 63, ug = tid >> 8;
  const int ux = (pos >> 4) - 1, uy = ((pos >> 2) & 3) - 1, uz = (pos & 3) - 1;
  const int l_slot = ((ux >> 1) + 1) * 9 + ((uy >> 1) + 1) * 3 + ((uz >> 1) + 1);
  const int l_coff = 4 * (ux & 1) + 2 * (uy & 1) + (uz & 1);
  const int l_ch = c0 + 4 * f_;
  const int l_lds = 2 * ((f_ >> 1) * HS + ug * GS + (ux + 1) * XS + (uy + 1) * YS + (uz + 1)) +
                    (f_ & 1);  // in 8-byte units
  // Loads through buffer resources, one multiply and no branch each.  Groups
  // past the range read as row 0 (their results are not stored), absent rows
  // and channels past kk as zeros.
  const __amdgpu_buffer_rsrc_t rx_ = rsrc(x, BIG ? 0 : (uint32_t)(8 * ngroups * kk * 4));
  const bool dead = l_ch >= kk;
  int32_t nbn[NU];
  auto load_nb = [&](int t) {
    const int64_t gt = g0 + (int64_t)t * GPB;
    const int live = gt < g1 ? (int)std::min<int64_t>(GPB, g1 - gt) : 0;
    const __amdgpu_buffer_rsrc_t rn = rsrc(nbr + (live ? 27 * gt : 0), 108 * live);
#pragma unroll
    for (int i = 0; i < NU; ++i)
      nbn[i] = __builtin_amdgcn_raw_buffer_load_b32(rn, 4 * (27 * ug + l_slot) + 216 * i, 0, 0);
  };
  v4f rxs[2][NU];
  auto load_x = [&](v4f (&rx)[NU]) {
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if constexpr (BIG) {  // rows of 4 GiB and more: 64-bit addresses
        rx[i] = v4f{0.f, 0.f, 0.f, 0.f};
        if (nbn[i] >= 0 && !dead)
          rx[i] = *reinterpret_cast<const v4f*>(x + (int64_t)(nbn[i] + l_coff) * kk + l_ch);
      } else {
        const uint32_t off = (uint32_t)(nbn[i] + l_coff) * (uint32_t)(4 * kk) + 4 * l_ch;
        rx[i] = __builtin_bit_cast(
            v4f, __builtin_amdgcn_raw_buffer_load_b128(rx_, nbn[i] < 0 || dead ? ~0u : off, 0, 0));
      }
    }
  };
  auto store_x = [&](v4u* buf, const v4f (&rx)[NU]) {
    v2u* b2 = reinterpret_cast<v2u*>(buf);
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      v2u s[3];
      oc::s3_split4(sk, rx[i], s);
#pragma unroll
      for (int p = 0; p < 3; ++p) b2[l_lds + 2 * (p * PS + 2 * i * GS)] = s[p];
    }
  };

  // reads: lane (li, q) supplies row li of a row block: child li & 7 of group
  // 2 rb + (li >> 3); bases by what the pair's second tap (q >= 2) adds
  int base[4];
  {
    const int c = li & 7, sec = q >> 1;
    const int b = (q & 1) * HS + (2 * wm * RB + (li >> 3)) * GS + (c >> 2) * XS +
                  ((c >> 1) & 1) * YS + (c & 1);
    base[0] = b + sec * XS, base[1] = b + sec * YS, base[2] = b + sec, base[3] = b;
  }

  load_nb(0);
  load_x(rxs[0]);
  load_nb(1);
  v4u wr[NST / 2][3];
  {
    const int n = n0 + li, c = c0 + 8 * (q & 1);
#pragma unroll
    for (int s = 0; s < NST / 2; ++s) {
      const Pair p0 = pair_of(s), p1 = pair_of(s + NST / 2);
      const int k = th == 0 ? (q < 2 ? p0.a : p0.b) : (q < 2 ? p1.a : p1.b);
      v4f a = {0.f, 0.f, 0.f, 0.f}, b = a;
      if (k >= 0 && n < nn) {
        if constexpr (FLIP) {
          const float* p = w + ((int64_t)(26 - k) * nn + n) * kk + c;
          if (c < kk) a = *reinterpret_cast<const v4f*>(p);
          if (c + 4 < kk) b = *reinterpret_cast<const v4f*>(p + 4);
        } else {
          const float* p = w + ((int64_t)k * kk + c) * nn + n;
          if (c < kk) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = p[(int64_t)j * nn];
          }
          if (c + 4 < kk) {
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = p[(int64_t)(j + 4) * nn];
          }
        }
      }
      const oc::Split8 sp = oc::s3_split8(sk, a, b);
#pragma unroll
      for (int p = 0; p < 3; ++p) wr[s][p] = sp.p[p];
    }
  }

  // NB row blocks from block rb0 of the tile on, tap half H.  A unit is a step
  // of P row blocks, whose products are taken in turn, so that one need not
  // wait for the one before it (with one block, two sums do that); the reads
  // of the D-th next unit are issued before a unit's MFMAs.
  auto compute = [&](const v4u* buf, int rb0, auto half, auto nbt, v4f* acc) __attribute__((always_inline)) {
    constexpr int NB = decltype(nbt)::value, S0 = decltype(half)::value * (NST / 2);
    constexpr int P = NB >= 2 ? 2 : 1, U = NST / 2 * NB / P, D = P == 1 ? 2 : 1;
    const v4u* bb = buf + 2 * rb0 * GS;
    v4u f[D + 1][P][3];
    auto rd = [&](int u, int r, int p) {  // part p of row block r of unit u
      const int s = S0 + u * P / NB, r0 = u * P % NB;
      const int kind = s < 9 ? 0 : s < 12 ? 1 : s == 12 ? 2 : 3;
      f[u % (D + 1)][r][p] = bb[base[kind] + tap_off(pair_of(s).a) + 2 * (r0 + r) * GS + p * PS];
    };
    v4f c[NB], d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < NB; ++r) c[r] = d;
#pragma unroll
    for (int u = 0; u < D; ++u)
#pragma unroll
      for (int i = 0; i < 3 * P; ++i) rd(u, i / 3, i % 3);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        // one read, then the MFMAs it is issued beside
        if (u + D < U && (P == 2 || i % 2 == 0)) rd(u + D, P == 2 ? i / 3 : 0, P == 2 ? i % 3 : i / 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < P; ++r) {
          v4f& t = P == 1 && i % 2 == 0 ? d : c[u * P % NB + r];
          t = oc::s3_product(i, wr[u * P / NB], f[u % (D + 1)][r], t);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (P == 1) c[0] += d;
#pragma unroll
    for (int r = 0; r < NB; ++r) acc[r] = c[r];
  };
  typedef std::integral_constant<int, 0> H0;
  typedef std::integral_constant<int, 1> H1;
  typedef std::integral_constant<int, RB> All;
  typedef std::integral_constant<int, 1> One;

  const int64_t nrows = 8 * ngroups;
  const bool split = gridDim.z > 1;
  float* dst = split ? part + (int64_t)blockIdx.z * nrows * nn : out;
  // What is not finite is worked out again with fp32 MFMAs (16x16x4), by the
  // whole wave: lane l's four values are output channels n0 + 4 q .. + 3 of row
  // li of a row block, a row of group g.  Step j of a tap takes the channels
  // c0 + 4 q + j, so that a lane's four are one load of x.  The loads of three
  // taps are in flight together; absent neighbours read as zeros.
  // All NaN, 24 -> 40 channels on 12924 groups: 350 us (67 with ordinary values;
  // 106 in the fp32 kernel that this one replaced; 10600 with a serial sum per
  // value); 16 -> 16 on 9205: 41 (14; 21; 1030).
  auto mend = [&](int64_t g, v4f& v) __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // nothing of this is worked out ahead of the tile loop
    const int c = ln & 7, ch = c0 + 4 * (ln >> 4), n = n0 + (ln & 15);
    const int32_t* nb = nbr + 27 * (g < g1 ? g : g0);
    const __amdgpu_buffer_rsrc_t rw = rsrc(w, (uint32_t)(27 * kk * nn * 4));
    const uint32_t ow = n >= nn || ch >= kk ? ~0u : FLIP ? 4 * (n * kk + ch) : 4 * (ch * nn + n);
    v4f s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int kxy = 0; kxy < 9; ++kxy) {
      const int vx = (c >> 2) + kxy / 3 - 1, vy = ((c >> 1) & 1) + kxy % 3 - 1;
      v4f a[3], b[3];
#pragma unroll
      for (int kz = 0; kz < 3; ++kz) {
        const int vz = (c & 1) + kz - 1, k = 3 * kxy + kz;
        const int32_t e = nb[((vx >> 1) + 1) * 9 + ((vy >> 1) + 1) * 3 + (vz >> 1) + 1];
        const int64_t row = e + 4 * (vx & 1) + 2 * (vy & 1) + (vz & 1);
        if constexpr (BIG) {
          b[kz] = v4f{0.f, 0.f, 0.f, 0.f};
          if (e >= 0 && ch < kk) b[kz] = *reinterpret_cast<const v4f*>(x + row * kk + ch);
        } else {
          const uint32_t off = (uint32_t)row * (uint32_t)(4 * kk) + 4 * ch;
          b[kz] = __builtin_bit_cast(
              v4f, __builtin_amdgcn_raw_buffer_load_b128(rx_, e < 0 || ch >= kk ? ~0u : off, 0, 0));
        }
        if constexpr (FLIP) {
          a[kz] = __builtin_bit_cast(
              v4f, __builtin_amdgcn_raw_buffer_load_b128(rw, ow, 4 * (26 - k) * nn * kk, 0));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            a[kz][j] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rw, ow, 4 * (k * kk + j) * nn, 0));
        }
      }
#pragma unroll
      for (int kz = 0; kz < 3; ++kz)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kz][j], b[kz][j], s, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (!(fabsf(v[j]) < __builtin_inff())) v[j] = s[j];
  };
  // row block rb of the tile that starts at group gt
  auto store_rb = [&](int64_t gt, int rb, v4f v, int32_t pr) __attribute__((always_inline)) {
    if constexpr (POOL) {
      // through the wave's LDS area: lane o < 32 pools group o/16 of the
      // row block in channel n0 + o%16
      if (relu) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = fmaxf(v[j], 0.f);
      }
      float* pl = &PL[wv][0];
      oc::pool_put(pl, v, lane);
      uint32_t sw;
      const float m = oc::pool_scan(pl, lane, sw);
      const int c = n0 + (lane & 15);
      const int64_t g = gt + 2 * rb + ((lane >> 4) & 1);
      if (lane < 32 && c < nn && g < g1) {
        out[(int64_t)pr * nn + c] = m;
        psw[g * nn + c] = (uint8_t)sw;
      }
      return;
    }
    const int n = n0 + 4 * (lane & 3);
    const int64_t row = 8 * gt + 16 * rb + (lane >> 2);
    v4f sv = oc::store_order(v, lane);
    if (n < nn && row < 8 * g1) {
      if (!split && relu) {
#pragma unroll
        for (int j = 0; j < 4; ++j) sv[j] = fmaxf(sv[j], 0.f);
      }
      *reinterpret_cast<v4f*>(dst + row * nn + n) = sv;
    }
  };

  v4f acc[RB];
  int32_t prq[RB];
  // the wave's row blocks of tile t, the first at group g0 + t GPB + 2 wm RB
  auto multiply = [&](int t, auto half) __attribute__((always_inline)) {
    const v4u* buf = X + (t & 1) * BUFC;
    const int64_t left = g1 - g0 - (int64_t)t * GPB - 2 * wm * RB;  // groups from there on
    if (left > 2 * (RB - 1)) {
      compute(buf, 0, half, All{}, acc);
    } else {
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        acc[r] = v4f{0.f, 0.f, 0.f, 0.f};
        if (r < RB - 1 && left > 2 * r) compute(buf, r, half, One{}, acc + r);
      }
    }
  };
  auto finish = [&](int t) __attribute__((always_inline)) {  // first half: write tile t
    const v4f* ex = &EX[t & 1][wv][lane];
    const int64_t gt = g0 + (int64_t)t * GPB;
    v4f v[RB];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      v[r] = (acc[r] + ex[64 * r]) * oc::kSplitDown;
      bad |= oc::s3_bad(v[r]);
    }
    if (__builtin_expect(__any(bad), 0)) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (__any(oc::s3_bad(v[r]))) mend(gt + 2 * (wm * RB + r) + (li >> 3), v[r]);
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) store_rb(gt, wm * RB + r, v[r], POOL ? prq[r] : 0);
  };
  // tile t + 1 to LDS, tile t + 3 on its way
  auto stage = [&](int t, v4f (&rx)[NU]) {
    if (t + 1 < T) store_x(X + ((t + 1) & 1) * BUFC, rx);
    if (t + 3 < T) {
      load_x(rx);
      load_nb(t + 4);
    }
  };
  auto phase = [&](int t, v4f (&rx)[NU]) __attribute__((always_inline)) {
    lds_barrier();
    if (th == 0) {
      if (t > 0) finish(t - 1);
      if constexpr (POOL) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const int64_t g = g0 + (int64_t)t * GPB + 2 * (wm * RB + r) + ((lane >> 4) & 1);
          prq[r] = g < g1 ? prow[g] : -1;
        }
      }
      stage(t, rx);
      multiply(t, H0{});
    } else {
      multiply(t, H1{});
      v4f* ex = &EX[t & 1][wv][lane];
#pragma unroll
      for (int r = 0; r < RB; ++r) ex[64 * r] = acc[r];
      stage(t, rx);
    }
  };

  load_x(rxs[1]);  // groups past the range read as row 0
  load_nb(2);
  store_x(X, rxs[0]);
  load_x(rxs[0]);
  load_nb(3);
  for (int t = 0; t < T; t += 2) {
    phase(t, rxs[1]);
    if (t + 1 < T) phase(t + 1, rxs[0]);
  }
  lds_barrier();
  if (th == 0) finish(T - 1);
}

template <int WN, int GPB, bool FLIP, bool POOL, bool BIG>
void launch_sp3b(const oc_octree* t, int l, int splits, const float* x, int kk, const float* w, int nn,
            float* out, int relu, float* part, const oc::Sp3Pool* po, hipStream_t s) {
  const auto kernel = k_conv_sp3<WN, GPB, FLIP, POOL, BIG>;
  const int64_t G = t->M[l - 1];
  const int64_t gy = oc::cdiv(nn, 16 * WN), gyz = gy * splits;
  // one resident workgroup per CU, each over a contiguous range of groups
  int64_t px = std::min<int64_t>(G, std::max<int64_t>(1, (int64_t)oc::cu_count() / gyz));
  if (px >= 8) px -= px % 8;
  const dim3 grid((unsigned)px, (unsigned)gy, (unsigned)splits);
  oc::launch_main(kernel, grid, dim3(TB), s, (const int32_t*)t->nbr[l], G, x, kk, w, nn,
                  POOL ? po->y : out, relu, part, (const int32_t*)t->rows[l - 1],
                  (const int32_t*)t->labels[l - 1], t->N[l - 1],
                  POOL ? po->sw : (uint8_t*)nullptr);
}

template <int WN, int GPB, bool FLIP, bool POOL>
void launch_sp3(const oc_octree* t, int l, int splits, const float* x, int kk, const float* w,
                int nn, float* out, int relu, float* part, const oc::Sp3Pool* po, hipStream_t s) {
  if (rows_big(t, l, kk))
    launch_sp3b<WN, GPB, FLIP, POOL, true>(t, l, splits, x, kk, w, nn, out, relu, part, po, s);
  else
    launch_sp3b<WN, GPB, FLIP, POOL, false>(t, l, splits, x, kk, w, nn, out, relu, part, po, s);
}

// ---------------------------------------------------------------------------
// Weight gradient, K = 3, cin >= 16 (k_conv_dws):
//   dW[k][c][n] = sum over octants i of x[nb(i,k)][c] dY[i][n],
// products from three bf16 parts.  The MFMA (16x16x32) reduces over the octants
// of four sibling groups: lane group q = l / 16 supplies the eight children of
// group q, for A (16 channels) and B (16 columns) alike.  Both are staged as
// rows of channels and read with transposing LDS loads (ds_read_b64_tr_b16:
// lane i of a lane group gets channel i of the four rows whose 8-byte quarters
// the group's lanes name), two per operand part, one per x-bit of the children.
//
// A workgroup (chunk, tile) owns 16 channels by 16 NBN columns and a chunk of
// groups.  It is two halves of four waves; the halves take alternate stages of
// four groups, each in two LDS buffers of its own, and a half's waves take taps
// w, w + 4, ...  One barrier per stage: between two of them stage s is
// multiplied, stage s + 1, loaded a stage earlier, is split and stored, and
// stage s + 2 is loaded.  Half 0 stores first and half 1 multiplies first, so
// that each SIMD has one wave of either kind of work.  At the end the halves'
// sums meet through LDS and go to part[chunk][27 cin][cout].
//
// LDS: part p, group g, position (x, y, z) is the 32-byte row 264 p + 66 g +
// 16 x + 4 y + z; the four rows of a transposing load and those of the next
// group are then distinct mod 8, which is all 64 banks.  dY: part, group, child
// rows of 32 NBN bytes, groups padded to the same end.
//
// What is not finite is worked out again, wave by wave, with fp32 MFMAs: 243 us
// for all NaN, 24 -> 40 channels on 12924 groups (85 with ordinary values, 112 in
// the kernel before).
//
// Measured on an MI355X (before: an fp32 16x16x4 kernel of the same tiles):
// 16 -> 16 channels on 211730 groups of depth 8 208 us, 113 TFLOP/s of fp32
// products, and 16 -> 64 on 67121 of depth 6 172 us, 173; the whole 24 -> 40
// layer of 5 shapes at depth 6, three passes, 224 -> 182 us.
// With 16 columns the split and store of x, which two halves' waves share with
// 84 MFMAs each, bound it; with 32 the MFMAs do.
template <int NBN, bool BIG>
__global__ __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_dws(
    const int32_t* __restrict__ nbr, int64_t ngroups, int64_t gchunk, const float* __restrict__ x,
    int cin, const float* __restrict__ dy, int cout, float* __restrict__ part) {
  constexpr int GS = 4, NJ = 7, HT = TB / 2;  // groups a stage, taps a wave, threads a half
  constexpr int BN = 16 * NBN;
  constexpr int XG = 66 * 32, XP = GS * XG;                                // bytes
  constexpr int YG = 8 * BN * 2 + (NBN == 1 ? 128 : 32), YP = GS * YG;
  constexpr int BUF = 3 * (XP + YP);
  constexpr int NRED = NJ * NBN * 4 * 64 * 16;
  constexpr int NSM = 4 * BUF > NRED ? 4 * BUF : NRED;
  static_assert(XG % 16 == 0 && YG % 16 == 0 && NSM <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(16))) char smem[NSM];

  const int tid = threadIdx.x & (HT - 1), lane = tid & 63;
  const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / HT);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, q = lane >> 4;
  const int nCB = (cin + 15) / 16;
  const int c0 = 16 * (int)(blockIdx.y % nCB), n0 = BN * (int)(blockIdx.y / nCB);
  const int64_t gb = (int64_t)blockIdx.x * gchunk;
  const int64_t ge = gb + gchunk < ngroups ? gb + gchunk : ngroups;
  if (gb >= ge) return;  // uniform over the workgroup
  const int ng = (int)(ge - gb);
  const int nsub = (ng + 2 * GS - 1) / (2 * GS);  // stages of a half
  char* const mine = smem + half * 2 * BUF;

  const oc::SplitK sk = oc::s3_consts();
  // x staging: thread -> position, channel quad, every group of the stage
  const int f = tid & 3, pos = tid >> 2;
  const int ux = (pos >> 4) - 1, uy = ((pos >> 2) & 3) - 1, uz = (pos & 3) - 1;
  const int slot = ((ux >> 1) + 1) * 9 + ((uy >> 1) + 1) * 3 + ((uz >> 1) + 1);
  const int coff = 4 * (ux & 1) + 2 * (uy & 1) + (uz & 1);
  const int ch = c0 + 4 * f;
  const int lx = pos * 32 + f * 8;
  // dY staging: thread -> row of the stage, column quad (8 GS 4 NBN <= HT)
  const int yr = tid / (4 * NBN), yf = tid % (4 * NBN), yn = n0 + 4 * yf;
  const bool yon = yr < 8 * GS;
  const int ly = 3 * XP + (yr >> 3) * YG + (yr & 7) * BN * 2 + yf * 8;
  // buffer resources relative to the chunk: what lies past it reads as zero
  const __amdgpu_buffer_rsrc_t rn = rsrc(nbr + 27 * gb, 108u * (uint32_t)ng);
  const __amdgpu_buffer_rsrc_t rx_ = rsrc(x, BIG ? 0 : (uint32_t)(8 * ngroups * cin * 4));
  const __amdgpu_buffer_rsrc_t ry_ =
      rsrc(dy + 8 * gb * cout, BIG ? 0 : (uint32_t)(8 * (int64_t)ng * cout * 4));

  int32_t nb[GS];
  auto first = [&](int s) { return (2 * s + half) * GS; };  // first group of stage s
  auto load_nb = [&](int s) {
#pragma unroll
    for (int i = 0; i < GS; ++i) {
      const int g = first(s) + i;  // groups past the chunk: absent
      const int32_t v = __builtin_amdgcn_raw_buffer_load_b32(rn, 4 * slot, 108 * (g < ng ? g : 0), 0);
      nb[i] = v;
    }
  };
  v4f rx[GS], ry;
  auto load = [&](int s) {
#pragma unroll
    for (int i = 0; i < GS; ++i) {
      const bool live = first(s) + i < ng && nb[i] >= 0 && ch < cin;
      if constexpr (BIG) {
        rx[i] = v4f{0.f, 0.f, 0.f, 0.f};
        if (live) rx[i] = *reinterpret_cast<const v4f*>(x + (int64_t)(nb[i] + coff) * cin + ch);
      } else {
        const uint32_t off = (uint32_t)(nb[i] + coff) * (uint32_t)(4 * cin) + 4 * ch;
        rx[i] = __builtin_bit_cast(
            v4f, __builtin_amdgcn_raw_buffer_load_b128(rx_, live ? off : ~0u, 0, 0));
      }
    }
    const bool live = yon && first(s) + (yr >> 3) < ng && yn < cout;
    if constexpr (BIG) {
      ry = v4f{0.f, 0.f, 0.f, 0.f};
      if (live)
        ry = *reinterpret_cast<const v4f*>(dy + (8 * (gb + first(s)) + yr) * (int64_t)cout + yn);
    } else {
      const uint32_t off = (uint32_t)(8 * first(s) + yr) * (uint32_t)(4 * cout) + 4 * yn;
      ry = __builtin_bit_cast(
          v4f, __builtin_amdgcn_raw_buffer_load_b128(ry_, live ? off : ~0u, 0, 0));
    }
  };
  auto store = [&](int s) {
    char* b = mine + (s & 1) * BUF;
#pragma unroll
    for (int i = 0; i < GS; ++i) {
      v2u p[3];
      oc::s3_split4(sk, rx[i], p);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<v2u*>(b + lx + k * XP + i * XG) = p[k];
    }
    if (yon) {
      v2u p[3];
      oc::s3_split4(sk, ry, p, half ? -oc::kSplitUp : oc::kSplitUp);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<v2u*>(b + ly + k * YP) = p[k];
    }
  };

  // reads: lane li names the 8-byte quarter li & 3 of row (child) 4 hh + (li >> 2)
  const int r4 = li >> 2, tq = li & 3;
  int ax[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int tap = wave + 4 * j < 27 ? wave + 4 * j : 0;
    ax[j] = q * XG + tq * 8 + 32 * (16 * (tap / 9) + 4 * (tap / 3 % 3 + (r4 >> 1)) + tap % 3 + (r4 & 1));
  }
  const int by = 3 * XP + q * YG + r4 * BN * 2 + tq * 8;
  v4f acc[NJ][NBN];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int n = 0; n < NBN; ++n) acc[j][n] = v4f{0.f, 0.f, 0.f, 0.f};

  // P taps a unit, so that two sums at least are in turn; the reads of the
  // next unit are issued before a unit's MFMAs.  A stage's six products are
  // summed from zero and then added to the running sum, which is rounded once
  // a stage that way, to nearest: the MFMA adding all six to it was measured to
  // leave six times the fp32 kernel's error (3.8e-6 of dW at 218768 groups, 16 ->
  // 16).  The MFMA itself cuts its sums off, always downwards it seems: with dY
  // as it is in both halves, 1.5e-6 was left, growing with the octants as a bias
  // does.  Half 1 therefore takes -dY, so that the two halves' biases cancel:
  // 2.1e-7, and 1.8e-6 for 256 -> 256 on 159111 groups (fp32 kernel 1.0e-5).  (Tap
  // 27 of wave 3 reads tap 0's rows; its sum is dropped.)
  auto multiply = [&](int s) {
    constexpr int P = NBN == 1 ? 2 : 1, U = (NJ + P - 1) / P;
    const char* b = mine + (s & 1) * BUF;
    v4u bq[NBN][3], a[2][P][3];
#pragma unroll
    for (int n = 0; n < NBN; ++n)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        bq[n][k] = tr2(b + by + k * YP + n * 32, 4 * BN * 2);
    auto rd = [&](int u) {
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (u * P + i < NJ) {
#pragma unroll
          for (int k = 0; k < 3; ++k) a[u & 1][i][k] = tr2(b + ax[u * P + i] + k * XP, 16 * 32);
        }
    };
    v4f t[2][P][NBN];
    auto add = [&](int u) {
#pragma unroll
      for (int r = 0; r < P; ++r)
        if (u * P + r < NJ) {
#pragma unroll
          for (int n = 0; n < NBN; ++n) acc[u * P + r][n] += t[u & 1][r][n];
        }
    };
    rd(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u + 1 < U) rd(u + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int r = 0; r < P; ++r)
          if (u * P + r < NJ) {
#pragma unroll
            for (int n = 0; n < NBN; ++n)
              t[u & 1][r][n] = oc::s3_product(i, a[u & 1][r], bq[n],
                                              i == 0 ? v4f{0.f, 0.f, 0.f, 0.f} : t[u & 1][r][n]);
          }
      if (u > 0) add(u - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    add(U - 1);
  };

  load_nb(0);
  load(0);
  load_nb(1);
  store(0);
  load(1);
  load_nb(2);
  auto stage = [&](int s) {  // stage s to LDS, s + 1 on its way
    if (s >= nsub) return;
    store(s);
    load(s + 1);
    load_nb(s + 2);
  };
  for (int s = 0; s < nsub; ++s) {
    lds_barrier();
    if (half == 0) {
      stage(s + 1);
      multiply(s);
    } else {
      multiply(s);
      stage(s + 1);
    }
  }

  bool bad = false;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int n = 0; n < NBN; ++n) bad |= oc::s3_bad(acc[j][n]);
  if (__builtin_expect(__any(bad), 0)) {  // this wave's sums again, in plain fp32
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int n = 0; n < NBN; ++n) acc[j][n] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < nsub * GS; ++i) {  // a sibling group: its eight children in two steps
      const int gl = first(i / GS) + i % GS;
      if (gl >= ng) break;
      int32_t e[2][NJ];
      float av[2][NJ], bv[2][NBN];
#pragma unroll
      for (int h = 0; h < 2; ++h)  // child 4 h + q: the lane group's
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int tap = wave + 4 * j < 27 ? wave + 4 * j : 0;
          const int vx = h + tap / 9 - 1, vy = (q >> 1) + tap / 3 % 3 - 1, vz = (q & 1) + tap % 3 - 1;
          const int sl = ((vx >> 1) + 1) * 9 + ((vy >> 1) + 1) * 3 + (vz >> 1) + 1;
          const int32_t v = __builtin_amdgcn_raw_buffer_load_b32(rn, 4 * sl, 108 * gl, 0);
          e[h][j] = v < 0 ? v : v + 4 * (vx & 1) + 2 * (vy & 1) + (vz & 1);
        }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int n = 0; n < NBN; ++n) {
          const int col = n0 + 16 * n + li;
          bv[h][n] = col < cout ? dy[(8 * (gb + gl) + 4 * h + q) * cout + col] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bool live = e[h][j] >= 0 && c0 + li < cin;
          if constexpr (BIG) {
            av[h][j] = live ? x[(int64_t)e[h][j] * cin + c0 + li] : 0.f;
          } else {
            const uint32_t off = (uint32_t)e[h][j] * (uint32_t)(4 * cin) + 4 * (c0 + li);
            av[h][j] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rx_, live ? off : ~0u, 0, 0));
          }
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int n = 0; n < NBN; ++n)
            acc[j][n] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(av[h][j], bv[h][n], acc[j][n], 0, 0, 0);
    }
  } else {
    const float down = half ? -oc::kSplitDown : oc::kSplitDown;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int n = 0; n < NBN; ++n) acc[j][n] *= down;
  }

  // halves add their sums: tap j goes to half j < JH ? 0 : 1
  constexpr int JH = (NJ + 1) / 2;
  v4f* red = reinterpret_cast<v4f*>(smem);
  __syncthreads();  // the last stage's LDS reads are done
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if ((j < JH) != (half == 0))
#pragma unroll
      for (int n = 0; n < NBN; ++n) red[((j * NBN + n) * 4 + wave) * 64 + lane] = acc[j][n];
  __syncthreads();
  float* pp = part + (int64_t)blockIdx.x * 27 * cin * cout;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int tap = wave + 4 * j;
    if (tap >= 27 || (j < JH) != (half == 0)) continue;
#pragma unroll
    for (int n = 0; n < NBN; ++n) {
      const v4f v = acc[j][n] + red[((j * NBN + n) * 4 + wave) * 64 + lane];
      const int col = n0 + 16 * n + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // row 4 q + r of the product: the channel
        const int c = c0 + 4 * q + r;
        if (c < cin && col < cout) pp[((int64_t)tap * cin + c) * cout + col] = v[r];
      }
    }
  }
}

template <int NBN>
void launch_dws(const oc_octree* t, int l, int64_t gchunk, int64_t nchunks, const float* x,
                int cin, const float* dy, int cout, float* part, hipStream_t s) {
  const bool big = rows_big(t, l, std::max(cin, cout));
  const auto kernel = big ? k_conv_dws<NBN, true> : k_conv_dws<NBN, false>;
  const dim3 grid((unsigned)nchunks, (unsigned)(oc::cdiv(cin, 16) * oc::cdiv(cout, 16 * NBN)));
  oc::launch_main(kernel, grid, dim3(TB), s, (const int32_t*)t->nbr[l], t->M[l - 1], gchunk, x, cin,
                  dy, cout, part);
}

}  // namespace

namespace oc {

Sp3Cfg sp3_pick(int64_t G, int kk, int nn) {
  Sp3Cfg c;
  c.wn = nn <= 16 ? 1 : nn <= 32 ? 2 : 4;
  c.splits = (int)cdiv(kk, 16);
  // Tile size: the least time for the longest range of groups (a workgroup per
  // CU), counting a wave's row blocks plus a fixed cost per tile (barrier,
  // loads, stores) of one row block.
  const int64_t gyz = cdiv(nn, 16 * c.wn) * c.splits;
  const int64_t ng = cdiv(G, std::max<int64_t>(1, (int64_t)cu_count() / gyz));
  const int wm = 4 / c.wn;
  double best = 1e30;
  c.gpb = 8;
  for (int gpb = 8; gpb / 2 >= wm; gpb /= 2) {
    const int64_t full = ng / gpb, tail = ng - full * gpb;
    const double cost = full * (gpb / 2 / wm + 1.0) +
                        (tail > 0 ? (double)cdiv(cdiv(tail, 2), wm) + 1.0 : 0.0);
    if (cost < best - 1e-9) best = cost, c.gpb = gpb;
  }
  return c;
}

#define OC_SP3_LIST(X) X(1, 8) X(2, 8) X(2, 4) X(4, 8) X(4, 4) X(4, 2)

void sp3_launch(const oc_octree* t, int l, const Sp3Cfg& c, bool flip, const float* x, int kk,
                const float* w, int nn, float* out, int relu, float* part, const Sp3Pool* pool,
                hipStream_t s) {
#define OC_SP3(WN_, GPB_)                                                                       \
  if (c.wn == WN_ && c.gpb == GPB_) {                                                           \
    if (flip)                                                                                   \
      launch_sp3<WN_, GPB_, true, false>(t, l, c.splits, x, kk, w, nn, out, relu, part, pool, s);   \
    else if (pool && c.splits == 1)                                                             \
      launch_sp3<WN_, GPB_, false, true>(t, l, c.splits, x, kk, w, nn, out, relu, part, pool, s);   \
    else                                                                                        \
      launch_sp3<WN_, GPB_, false, false>(t, l, c.splits, x, kk, w, nn, out, relu, part, pool, s);  \
    return;                                                                                     \
  }
  OC_SP3_LIST(OC_SP3)
#undef OC_SP3
}

void sp3_name(const oc_octree* t, int l, const Sp3Cfg& c, bool flip, bool pooled, int kk, char* buf,
              size_t n) {
  const char* const tf[2] = {"false", "true"};
  snprintf(buf, n, "k_conv_sp3<%d, %d, %s, %s, %s>", c.wn, c.gpb, tf[flip],
           tf[pooled && c.splits == 1], tf[rows_big(t, l, kk)]);
}

void dws_launch(const oc_octree* t, int l, int nbn, int64_t gchunk, int64_t nchunks, const float* x,
                int cin, const float* dy, int cout, float* part, hipStream_t s) {
  if (nbn == 1)
    launch_dws<1>(t, l, gchunk, nchunks, x, cin, dy, cout, part, s);
  else
    launch_dws<2>(t, l, gchunk, nchunks, x, cin, dy, cout, part, s);
}

void dws_name(const oc_octree* t, int l, int nbn, int cin, int cout, char* buf, size_t n) {
  snprintf(buf, n, "k_conv_dws<%d, %s>", nbn, rows_big(t, l, std::max(cin, cout)) ? "true" : "false");
}

}  // namespace oc
