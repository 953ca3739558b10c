// Rank selection on bit planes, for windows of at most a few hundred taps.
//
// A lane holds one bit of 32 output pixels in each of its registers, so one
// 32-bit logical instruction works on 32 pixels.  The median is found from
// its most significant bit down (radix selection by halves): for every tap
// of the window a mask M says for which of the 32 pixels the tap still
// agrees with all bits found so far.  Per bit plane b:
//   t = M & ~b        taps that agree and have a 0 here
//   C = sum of t      over the taps, in bit-sliced full adders (two
//                     three-input logical instructions per tap)
//   bit = k >= C      k: the rank left; where the bit is 1, k -= C
//   M = bit ? M & ~t : t
// about 4.6 instructions per tap and plane for 32 pixels, whatever the
// window's shape, the values or the rank; the tile engine (tile_engine.h)
// ranks a box and walks it instead, about 2000 per pixel.  Bound by the
// vector ALU: at 4096 x 4096 uint16, disc 5 / 8, 263 / 770 instructions per
// pixel at 82 / 87 % of the issue rate, 1.23 -> 0.138 / 1.06 -> 0.37 ms
// against the tile engine (uint8 disc 2 1.99 -> 0.027 ms, float32 disc 4
// 2.07 -> 0.19 ms); the LDS is busy 37 / 35 % of the time.
//
// The 32 pixels of a word are not neighbours: the output tile is cut into
// GX x GY = 4 x 8 sub-tiles of SX x SY pixels and bit b of word (x, y)
// belongs to pixel (x, y) of sub-tile (b % GX, b / GX).  A tap (dx, dy) then
// is the word (x + dx, y + dy), bits unmoved: no funnel shifts, only an LDS
// address.  The words cover a sub-tile grown by the window.
//
// Per workgroup: the tile's input box goes to LDS with the boundary rule
// applied (float keys already ordered); for each byte of the key, most
// significant first, the eight planes of every word are gathered from it
// (8x8 bit transposes in registers), the eight bits are selected, and the
// result bytes are transposed back into the box, whose byte of that
// significance is no longer read.  Last, the box's tile is written out.
//
// Windows of more taps than a lane has registers for (it keeps M and t
// of every tap) are split over G lanes: each counts its own share, the
// bit-sliced counts are added across the lanes, and all G lanes go on with
// the same bit.
#pragma once

#include <type_traits>
#include <utility>

#include "tile_common.h"

namespace mf {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(static_cast<F&&>(f));
  }
}

// Three-input logic (v_bitop3_b32): bit i of the table is the result where
// the operands are the bits of i (first operand: 4, second: 2, third: 1).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xe8);
}
// ~a & b | c & ~(a ^ b): the borrow of a - b - c
__device__ __forceinline__ uint32_t borrow3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x8e);
}
// s ? a : b
__device__ __forceinline__ uint32_t sel3(uint32_t s, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_bitop3_b32(s, a, b, 0xca);
}

constexpr int bit_length(int n) { return n == 0 ? 0 : 1 + bit_length(n >> 1); }

// Bit-sliced count of one-bit words, streamed: A[l], B[l] hold the words of
// weight 2^l waiting to be added.  K = number of words pushed to level l so
// far including this one: the first waits in A, an even one in B, and an odd
// one meets both in a full adder whose carry is push (K - 1) / 2 of level
// l + 1.  count_finish adds what is left; bit l of the count is then A[l].
template <int L, int K, int NL>
__device__ __forceinline__ void count_push(uint32_t x, uint32_t (&A)[NL], uint32_t (&B)[NL]) {
  if constexpr (K == 1) {
    A[L] = x;
  } else if constexpr (K % 2 == 0) {
    B[L] = x;
  } else {
    const uint32_t c = maj3(A[L], B[L], x);
    A[L] = xor3(A[L], B[L], x);
    count_push<L + 1, (K - 1) / 2>(c, A, B);
  }
}
template <int L, int K, int NL>
__device__ __forceinline__ void count_finish(uint32_t (&A)[NL], uint32_t (&B)[NL]) {
  if constexpr (K > 0) {
    if constexpr (K % 2 == 0) {
      const uint32_t c = A[L] & B[L];
      A[L] ^= B[L];
      count_push<L + 1, K / 2>(c, A, B);
    }
    count_finish<L + 1, K / 2>(A, B);
  }
}

// A[0 .. N) += the same number held by the lanes STEP apart that share the
// window (all of them end with the sum, N + 1 bits).
template <int STEP, int N, int NL>
__device__ __forceinline__ void count_merge(uint32_t (&A)[NL]) {
  uint32_t x[N], y[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = y[i] = A[i];
  if constexpr (STEP >= 16) {
    // copies first, then the swaps, which must not follow a copy of their
    // operands at once
#pragma unroll
    for (int i = 0; i < N; ++i) asm("v_mov_b32 %0, %1" : "=v"(x[i]) : "v"(A[i]));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const auto r = STEP == 32 ? __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false)
                                : __builtin_amdgcn_permlane16_swap(x[i], y[i], false, false);
      x[i] = r[0];
      y[i] = r[1];
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i)
      y[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)A[i], STEP == 8 ? 0x128 : 0x124, 0xf, 0xf,
                                                   false);   // row_ror
  }
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    A[i] = xor3(x[i], y[i], c);
    c = maj3(x[i], y[i], c);
  }
  A[N] = c;
}

// 8x8 bit transposes within the bytes: on entry byte c of x[i] holds a
// byte of item i + 8c; on return x[q] holds bit q of item b in its bit b.
// Its own inverse.
template <int S, uint32_t M>
__device__ __forceinline__ void transpose8_stage(uint32_t (&x)[8]) {
  static_for<0, 8>([&](auto ii) {
    constexpr int i = decltype(ii)::value;
    if constexpr ((i & S) == 0) {
      const uint32_t a = x[i], b = x[i + S];
      x[i] = sel3(M, a, b << S);
      x[i + S] = sel3(M, a >> S, b);
    }
  });
}
__device__ __forceinline__ void transpose8(uint32_t (&x)[8]) {
  transpose8_stage<4, 0x0f0f0f0fu>(x);
  transpose8_stage<2, 0x33333333u>(x);
  transpose8_stage<1, 0x55555555u>(x);
}

// 16 bytes at any element's address (rows start anywhere: unaligned vector
// accesses are in order for global memory on this target).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));
template <typename T>
__device__ __forceinline__ u32x4 load16(const T* p) {
  return *reinterpret_cast<const u32x4_any*>(p);
}
template <typename T>
__device__ __forceinline__ void store16(T* p, u32x4 v) {
  *reinterpret_cast<u32x4_any*>(p) = v;
}

// bytes s0 s1 s2 s3 (least significant first) of the eight bytes b:a, a low
template <int S0, int S1, int S2, int S3>
__device__ __forceinline__ uint32_t pick4(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, S0 | S1 << 8 | S2 << 16 | S3 << 24);
}

// 4x4 byte transpose: byte c of x[i] <-> byte i of x[c].
__device__ __forceinline__ void transpose4(uint32_t& x0, uint32_t& x1, uint32_t& x2, uint32_t& x3) {
  const uint32_t a = pick4<0, 4, 1, 5>(x0, x1), b = pick4<2, 6, 3, 7>(x0, x1);
  const uint32_t c = pick4<0, 4, 1, 5>(x2, x3), d = pick4<2, 6, 3, 7>(x2, x3);
  x0 = pick4<0, 1, 4, 5>(a, c);
  x1 = pick4<2, 3, 6, 7>(a, c);
  x2 = pick4<0, 1, 4, 5>(b, d);
  x3 = pick4<2, 3, 6, 7>(b, d);
}

// The box in LDS is kept as byte planes (one per byte of the key, least
// significant first).  put_chunk splits 16 bytes of keys over them (dst: the
// chunk's place in the first plane, aligned to its pixels); get_chunk is
// its inverse.
template <int KT>
__device__ __forceinline__ void put_chunk(unsigned char* dst, int plane, u32x4 v) {
  if constexpr (KT == KEY_U8) {
    *reinterpret_cast<u32x4*>(dst) = v;
  } else if constexpr (KT == KEY_U16) {
    *reinterpret_cast<u32x2*>(dst) =
        u32x2{pick4<0, 2, 4, 6>(v.x, v.y), pick4<0, 2, 4, 6>(v.z, v.w)};
    *reinterpret_cast<u32x2*>(dst + plane) =
        u32x2{pick4<1, 3, 5, 7>(v.x, v.y), pick4<1, 3, 5, 7>(v.z, v.w)};
  } else {
    uint32_t a = f32_to_key(v.x), b = f32_to_key(v.y), c = f32_to_key(v.z), d = f32_to_key(v.w);
    transpose4(a, b, c, d);
    *reinterpret_cast<uint32_t*>(dst) = a;
    *reinterpret_cast<uint32_t*>(dst + plane) = b;
    *reinterpret_cast<uint32_t*>(dst + 2 * plane) = c;
    *reinterpret_cast<uint32_t*>(dst + 3 * plane) = d;
  }
}
template <int KT>
__device__ __forceinline__ u32x4 get_chunk(const unsigned char* src, int plane) {
  if constexpr (KT == KEY_U8) {
    return *reinterpret_cast<const u32x4*>(src);
  } else if constexpr (KT == KEY_U16) {
    const u32x2 l = *reinterpret_cast<const u32x2*>(src);
    const u32x2 h = *reinterpret_cast<const u32x2*>(src + plane);
    return u32x4{pick4<0, 4, 1, 5>(l.x, h.x), pick4<2, 6, 3, 7>(l.x, h.x),
                 pick4<0, 4, 1, 5>(l.y, h.y), pick4<2, 6, 3, 7>(l.y, h.y)};
  } else {
    uint32_t a = *reinterpret_cast<const uint32_t*>(src);
    uint32_t b = *reinterpret_cast<const uint32_t*>(src + plane);
    uint32_t c = *reinterpret_cast<const uint32_t*>(src + 2 * plane);
    uint32_t d = *reinterpret_cast<const uint32_t*>(src + 3 * plane);
    transpose4(a, b, c, d);
    return u32x4{key_to_f32(a), key_to_f32(b), key_to_f32(c), key_to_f32(d)};
  }
}
template <int KT>
__device__ __forceinline__ void put_element(unsigned char* dst, int plane, uint32_t v) {
  if (KT == KEY_F32) v = f32_to_key(v);
  constexpr int ES = KT == KEY_U8 ? 1 : KT == KEY_U16 ? 2 : 4;
#pragma unroll
  for (int i = 0; i < ES; ++i) dst[i * plane] = (unsigned char)(v >> (8 * i));
}

// An element as it lies in the image.
template <int KT>
using BitsElem = typename std::conditional<
    KT == KEY_U8, uint8_t, typename std::conditional<KT == KEY_U16, uint16_t, uint32_t>::type>::type;

// One output tile.  All threads of the workgroup must call it.  P: tap pairs
// per lane (two adjacent taps of a window row are read together).
template <int KT, int G, int P, typename D>
__device__ __forceinline__ void bits_body(const D& a, int tile, unsigned char* smem) {
  using Geo = BitsGeo<G>;
  using T = BitsElem<KT>;
  constexpr int NT = Geo::NT, SX = Geo::SX, SY = Geo::SY, GX = Geo::GX, GY = Geo::GY;
  constexpr int TW = Geo::TW, TH = Geo::TH, ES = (int)sizeof(T);
  constexpr int LW = bit_length(2 * P);
  constexpr int LG = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : G == 8 ? 3 : 4;
  constexpr int LT = LW + LG;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  constexpr int EC = 16 / ES;   // elements of a 16-byte chunk
  const int W = a.ncols, H = a.nrows;
  const BitsLayout ly = bits_layout(SX, SY, W, H);
  const int pitch = ly.pitch, nw = ly.nw, RP = ly.rp, RH = ly.rh;
  const int BP = RP * RH;                                         // bytes of a byte plane
  uint32_t* pl = reinterpret_cast<uint32_t*>(smem);              // 8 planes of nw words
  unsigned char* box = smem + 32 * nw;                            // ES byte planes
  uint32_t* tab = reinterpret_cast<uint32_t*>(box + ES * BP);     // G x P tap pairs
  const int tx0 = (tile % a.tiles_x) * TW, ty0 = (tile / a.tiles_x) * TH;
  const int gx0 = tx0 + a.dx_min, gy0 = ty0 + a.dy_min;

  // tap pairs: LDS byte offset of the first tap's word, bits 30 and 31 =
  // first and second tap present; pair i goes to lane share i % G
  if (wid == 0) {
    for (int i = lane; i < G * P; i += 64) tab[i] = 0;
    const short2 s = a.spans[min(lane, H - 1)];
    const int len = lane < H ? (int)s.y - (int)s.x + 1 : 0;
    const int np = (len + 1) >> 1;
    int idx = (int)wave_inclusive_scan((uint32_t)np, lane) - np;
    for (int q = 0; q < np; ++q, ++idx)
      tab[(idx % G) * P + idx / G] =
          (uint32_t)(4 * (lane * pitch + (int)s.x - a.dx_min + 2 * q)) |
          (2 * q + 1 < len ? 0xc0000000u : 0x40000000u);
  }
  // the box, as far as the tile's pixels inside the image need it: 16-byte
  // chunks where the image has them, kLB in flight per thread (a chunk across
  // the image's edge is read shifted inside), then the columns outside the
  // image pixel by pixel
  {
    constexpr int kLB = KT == KEY_F32 ? 8 : 4;
    const T* img = static_cast<const T*>(a.img);
    const int BW = min(TW, a.w - tx0) + W - 1, BH = min(TH, a.h - ty0) + H - 1;
    int c0 = max(0, -gx0), c1 = min(BW, a.w - gx0);   // box columns inside the image
    if (c1 - c0 < EC) c1 = c0 = 0;                     // fewer than a chunk: all by pixel
    const int j0 = c0 / EC, nj = (c1 + EC - 1) / EC - j0, n = nj * BH;
    if (nj > 0) {
      const int sx = NT % nj, sy = NT / nj;
      int cj = t % nj, cy = t / nj;
      for (int e0 = t; e0 < n; e0 += kLB * NT) {
        u32x4 v[kLB];
        int at[kLB], row[kLB];
#pragma unroll
        for (int j = 0; j < kLB; ++j) {
          // (past the last chunk: the last row's again, not stored)
          row[j] = min(cy, BH - 1);
          at[j] = (j0 + cj) * EC;
          const int gy = remap(gy0 + row[j], a.h, a.boundary);
          v[j] = load16(img + (long long)gy * a.stride + gx0 + min(max(at[j], c0), c1 - EC));
          cj += sx;
          cy += sy;
          if (cj >= nj) {
            cj -= nj;
            cy += 1;
          }
        }
#pragma unroll
        for (int j = 0; j < kLB; ++j) {
          if (e0 + j * NT >= n) break;
          unsigned char* dst = box + row[j] * RP;
          if (at[j] >= c0 && at[j] + EC <= c1) {
            put_chunk<KT>(dst + at[j], BP, v[j]);
          } else {
            const int s = min(max(at[j], c0), c1 - EC);
#pragma unroll
            for (int i = 0; i < EC; ++i)
              put_element<KT>(dst + s + i, BP, ES == 4 ? v[j][i]
                                                       : (v[j][i * ES / 4] >> (8 * (i * ES % 4))) &
                                                             ((1u << (8 * (ES % 4))) - 1u));
          }
        }
      }
    }
    const int no = BW - (c1 - c0);
    if (no > 0) {
      constexpr int kPB = 4;
      for (int e0 = t; e0 < no * BH; e0 += kPB * NT) {
        uint32_t v[kPB];
        int at[kPB];
#pragma unroll
        for (int j = 0; j < kPB; ++j) {
          const int e = min(e0 + j * NT, no * BH - 1);   // (the last one again, same value)
          const int y = e / no, o = e - y * no, x = o < c0 ? o : o + (c1 - c0);
          const int gx = remap(gx0 + x, a.w, a.boundary), gy = remap(gy0 + y, a.h, a.boundary);
          v[j] = (uint32_t)img[(long long)gy * a.stride + gx];
          at[j] = y * RP + x;
        }
#pragma unroll
        for (int j = 0; j < kPB; ++j) put_element<KT>(box + at[j], BP, v[j]);
      }
    }
  }
  __syncthreads();

  // this lane's word and share of the window
  constexpr int WL = 64 / G;
  const int g = lane / WL, word = wid * WL + (lane % WL);
  const int wx = word % SX, wy = word / SX;
  // (word offsets of two pairs share a register: below 2^16 bytes, and one
  // dot product with (1, 0) or (0, 1) unpacks and adds)
  uint32_t M[2 * P], off2[(P + 1) / 2];
  static_for<0, P>([&](auto ip) {
    constexpr int p = decltype(ip)::value;
    const uint32_t e = tab[g * P + p];
    const uint32_t o = (e & 0xffffu) + (uint32_t)(4 * (wy * pitch + wx));
    off2[p / 2] = p % 2 ? off2[p / 2] | (o << 16) : o;
    M[2 * p] = (e & 0x40000000u) ? ~0u : 0u;
    M[2 * p + 1] = (e & 0x80000000u) ? ~0u : 0u;
  });
  uint32_t kk[LT];
#pragma unroll
  for (int i = 0; i < LT; ++i) kk[i] = ((a.rank >> i) & 1) ? ~0u : 0u;

  for (int kb = ES - 1; kb >= 0; --kb) {
    // planes of byte kb
    if (kb != ES - 1) __syncthreads();   // the previous byte's planes are done with
    // (four words side by side per thread: a box dword has a byte of each)
    for (int n = t; n < nw / 4; n += NT) {
      const int pq = pitch / 4, y = n / pq, x = (n - y * pq) * 4;
      const unsigned char* src = box + kb * BP + y * RP + x;
      uint32_t v[4][8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t d[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)   // pixels of sub-tile i + 8c
          d[c] = *reinterpret_cast<const uint32_t*>(src + ((i + 8 * c) / GX) * SY * RP + (i % GX) * SX);
        transpose4(d[0], d[1], d[2], d[3]);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c][i] = d[c];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) transpose8(v[c]);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        *reinterpret_cast<u32x4*>(pl + q * nw + 4 * n) = u32x4{v[0][q], v[1][q], v[2][q], v[3][q]};
    }
    __syncthreads();
    // select its eight bits
    uint32_t r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = 0;
    // LDS address of the plane
    uint32_t plane = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem +
                     (uint32_t)(7 * 4 * nw);
#pragma unroll 1
    for (int q = 7; q >= 0; --q, plane -= 4 * nw) {
      auto words = [&](int p) {
        const uint32_t at = __builtin_amdgcn_udot2(
            __builtin_bit_cast(u16x2, off2[p / 2]), p % 2 ? u16x2{0, 1} : u16x2{1, 0}, plane, false);
        return (const __attribute__((address_space(3))) uint32_t*)(size_t)at;
      };
      uint32_t tt[2 * P];
      uint32_t A[LT + 1], B[LT + 1];
      // kAhead reads in flight: left alone, the scheduler issues each read
      // right before its use and every pair waits for the LDS
      constexpr int kAhead = P < 6 ? P : 6;
      uint32_t w0[kAhead], w1[kAhead];
      auto fetch = [&](auto ip) {
        constexpr int p = decltype(ip)::value;
        const auto* w = words(p);
        w0[p % kAhead] = w[0];
        w1[p % kAhead] = w[1];
      };
      static_for<0, kAhead>(fetch);
      static_for<0, P>([&](auto ip) {
        constexpr int p = decltype(ip)::value;
        const uint32_t t0 = M[2 * p] & ~w0[p % kAhead], t1 = M[2 * p + 1] & ~w1[p % kAhead];
        if constexpr (p + kAhead < P) fetch(std::integral_constant<int, p + kAhead>{});
        __builtin_amdgcn_sched_barrier(0x6);   // ALU instructions may cross, reads not
        tt[2 * p] = t0;
        tt[2 * p + 1] = t1;
        count_push<0, 2 * p + 1>(t0, A, B);
        count_push<0, 2 * p + 2>(t1, A, B);
      });
      count_finish<0, 2 * P>(A, B);
      if constexpr (G >= 2) count_merge<32, LW>(A);
      if constexpr (G >= 4) count_merge<16, LW + 1>(A);
      if constexpr (G >= 8) count_merge<8, LW + 2>(A);
      if constexpr (G >= 16) count_merge<4, LW + 3>(A);
      // k - C, borrow set where k < C
      uint32_t d[LT], bw = 0;
#pragma unroll
      for (int i = 0; i < LT; ++i) {
        d[i] = xor3(kk[i], A[i], bw);
        bw = borrow3(kk[i], A[i], bw);
      }
#pragma unroll
      for (int i = 0; i < LT; ++i) kk[i] = sel3(bw, kk[i], d[i]);
      const uint32_t m = ~bw;
#pragma unroll
      for (int i = 7; i > 0; --i) r[i] = r[i - 1];
      r[0] = m;
      // M = m ? M & ~t : t
      if (kb == 0 && q == 0) break;   // the last bit: no more to agree with
#pragma unroll
      for (int i = 0; i < 2 * P; ++i)
        M[i] = __builtin_amdgcn_bitop3_b32(M[i], tt[i], m, 0x64);
    }
    // r[i] is now bit i of the byte: back to bytes (byte c of r[i]: sub-tile
    // i + 8c), exchanged among four lanes side by side so that lane j holds
    // sub-tile i + 8j of all four, and into the box's byte plane (pixel (x, y)
    // of the tile at box position (x, y)); the G lanes of a word write a
    // share each
    transpose8(r);
    const int j4 = lane & 3;
    const uint32_t p1 = j4 & 1 ? 0x03070105u : 0x06020400u, p2 = j4 & 2 ? 0x03020706u : 0x05040100u;
    unsigned char* dst = box + kb * BP + (wy + 2 * j4 * SY) * RP + (wx & ~3);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r[i], 0xb1, 0xf, 0xf, false);
      const uint32_t b1 = __builtin_amdgcn_perm(a1, r[i], p1);
      const uint32_t a2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b1, 0x4e, 0xf, 0xf, false);
      const uint32_t b2 = __builtin_amdgcn_perm(a2, b1, p2);
      if (G == 1 || (i % (G < 8 ? G : 8)) == g)
        *reinterpret_cast<uint32_t*>(dst + (i / GX) * SY * RP + (i % GX) * SX) = b2;
    }
  }
  __syncthreads();
  for (int e = t; e < TW / EC * TH; e += NT) {
    const int x = e % (TW / EC) * EC, y = e / (TW / EC);
    const int gx = tx0 + x, gy = ty0 + y;
    if (gx >= a.w || gy >= a.h) continue;
    const u32x4 v = get_chunk<KT>(box + y * RP + x, BP);
    T* out = static_cast<T*>(a.out) + (long long)gy * a.stride + gx;
    if (gx + EC <= a.w) {
      store16(out, v);
    } else {
#pragma unroll
      for (int i = 0; i < EC; ++i)
        if (gx + i < a.w) out[i] = (T)(v[i * ES / 4] >> (8 * (i * ES % 4)));
    }
  }
}

}  // namespace mf
