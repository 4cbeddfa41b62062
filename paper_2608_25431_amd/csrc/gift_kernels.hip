// gfx950 kernels for segmented, per-user AES-256-GCM and the owner check.
//
// Hot path (k_gcm_tiles): one workgroup of 1024 threads per CU, its waves one
// team or two, each team persistent over 2 MiB tiles.  Each lane handles one
// 16-byte block per row of its team (1024 or 512 blocks):
//   - AES-256-CTR keystream from four T-tables in LDS, each replicated 32x so
//     that lane l reads copy (l mod 32) and a wave's random lookups never
//     collide in a bank; one v_perm_b32 forms each lookup address;
//   - one coalesced 16-byte load, XOR, 16-byte store;
//   - GHASH by per-lane Horner with M = H^row: Y <- Y*M xor X, where the
//     multiply by the fixed M uses 32 nibble-indexed tables (8 KiB per user)
//     staged in LDS.
// Tiles are aligned to the END of their segment, so the block at distance d
// from the segment's last block contributes X*H^(d + 2) to the GHASH sum; a
// tile t contributes P_t * H^(t*T) with P_t = sum of X*H^(d_t + 2) over its
// own blocks (d_t: distance from the tile's end), and lane l of a full tile
// ends at distance (row - 1 - l) from the tile's end.  Each wave multiplies
// its lanes' sums by their powers (one generic multiply) and XORs the wave's
// sum into the tile's; the last wave of the team to do so finishes the tile,
// while the others are in the next one.  The expansion cuts some tiles into
// row pieces (every tile when a call has fewer tiles than teams, else up to
// one per team at the queue's tail), whose partials meet by XOR.  The wave that
// completes a segment's rows folds its tiles and writes its tag.
//
// Around it: k_prologue (first kernel of a call: staged tables from pinned
// host memory, owner check), k_small (segments up to 1 KiB),
// zero-fill, the paged-call helpers, per-token encryption and key setup.
#include <hip/hip_runtime.h>

#include <stddef.h>

#include <mutex>

#include "gift_device.hpp"
#include "gift_internal.hpp"

namespace gift {

__constant__ AesConst c_aes = make_aes_const();

constexpr int32_t kVerdictOk = 0, kVerdictAuthFail = 1, kVerdictOwnerMixed = 2;

// LDS of k_gcm_tiles: the GHASH tables of each team, the AES tables (T0/T1,
// then T2/T3, 64 KiB each), the state of each team.
constexpr uint32_t kGtabBytes = 8192;  // 32 x 16 x 16 B GHASH tables of M

// A tile's record in LDS.
struct TileInfo {
  uint32_t g, s, trow, user;  // queue entry
  int32_t verdict;
  uint32_t pad[3];
  SegDesc desc;
  uint32_t rk[64];  // round keys (60 used)
};
// The sum of a tile and how far its team is with it.
struct TileSum {
  uint32_t z[4];   // XOR of the waves' sums
  uint32_t rows;   // waves that have done their rows
  uint32_t done;   // waves whose sum is in z
  uint32_t pad[2];
};
constexpr uint32_t kSlots = 4;  // tiles of a team that can be under way at once
// How the waves of a team follow each other through its tiles k = 0, 1, ...
// (see k_gcm_tiles).
struct TeamState {
  TileInfo info[kSlots];
  TileSum sum[kSlots];
  uint32_t rec;    // k + 1 once the records of tiles 0..k are in LDS
  uint32_t mtab;   // k + 1 once the tables of M hold tile k's user
  uint32_t fin;    // k + 1 once tiles 0..k are finished
  uint32_t pad;
};
// Offsets, and what a team is, with TEAMS teams per workgroup.
template <int TEAMS>
struct Team {
  static constexpr uint32_t threads = kThreads / TEAMS, waves = threads / 64;
  static constexpr int rows = kRows * TEAMS;  // rows of `threads` blocks per tile
  static constexpr uint32_t lds_aes = TEAMS * kGtabBytes, lds_state = lds_aes + 131072;
  static constexpr uint32_t lds_bytes = lds_state + TEAMS * sizeof(TeamState);
  static_assert(lds_bytes <= 160u * 1024u, "LDS of a gfx950 workgroup");
};

// A segment's descriptor by scalar loads, s wave-uniform.
__device__ __forceinline__ SegDesc ld_uniform(const SegDesc* p) {
  union {
    uint32_t w[sizeof(SegDesc) / 4];
    SegDesc d;
  } u;
  const uniform_ptr q = to_uniform((const uint32_t*)p);
#pragma unroll
  for (uint32_t i = 0; i < sizeof(SegDesc) / 4; i++) u.w[i] = q[i];
  return u.d;
}

// Counters in LDS between the waves of one workgroup, which are all resident
// until they end, so a wait for work that another wave does without waiting
// for this one ends.  wave_arrive and wave_set publish the wave's LDS writes
// before the count; wave_wait orders its later LDS accesses after it.
__device__ __forceinline__ uint32_t wave_arrive(uint32_t* c) {  // returns the arrivals before this one
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  uint32_t n = 0;
  if ((threadIdx.x & 63u) == 0u) n = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return (uint32_t)__builtin_amdgcn_readfirstlane(n);
}
__device__ __forceinline__ void wave_set(uint32_t* c, uint32_t v) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if ((threadIdx.x & 63u) == 0u) __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wave_wait(const uint32_t* c, uint32_t v) {
  while ((int32_t)(__builtin_amdgcn_readfirstlane(
                       __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) - v) < 0)
    __builtin_amdgcn_s_sleep(1);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t lds32(const uint8_t* base, uint32_t off) {
  return *(const uint32_t*)(base + off);
}
__device__ __forceinline__ uint4 lds128(const uint8_t* base, uint32_t off) { return *(const uint4*)(base + off); }

// T-table address of byte k of w for lane copy L: (x << 8) | (lane*4) in the
// first 64 KiB region (T0 at +0, T1 at +128) or, with the 0x10000 bit taken
// from L, the second region (T2 at +0, T3 at +128).
#define GIFT_SEL_A(k) (0x0c0c0000u | ((4u + (k)) << 8))
#define GIFT_SEL_B(k) (0x0c020000u | ((4u + (k)) << 8))
#define GIFT_T0(w, k) lds32(tt, __builtin_amdgcn_perm((w), L, GIFT_SEL_A(k)))
#define GIFT_T1(w, k) lds32(tt + 128, __builtin_amdgcn_perm((w), L, GIFT_SEL_A(k)))
#define GIFT_T2(w, k) lds32(tt, __builtin_amdgcn_perm((w), L, GIFT_SEL_B(k)))
#define GIFT_T3(w, k) lds32(tt + 128, __builtin_amdgcn_perm((w), L, GIFT_SEL_B(k)))

// AES-256 rounds R0..13 and the final round on a state that has been through
// rounds 1..R0-1 already.
template <int R0>
__device__ __forceinline__ void aes_rounds_lds(uint32_t& s0, uint32_t& s1, uint32_t& s2, uint32_t& s3,
                                               const uint32_t* rk, const uint8_t* tt, uint32_t L) {
#pragma unroll
  for (int r = R0; r < 14; r++) {
    // The LDS is the bottleneck: a wave that is forming addresses and issuing
    // its reads runs at raised priority, so the LDS queue is refilled as soon
    // as possible, and drops back while it combines results.
    __builtin_amdgcn_s_setprio(2);
    // all 16 lookups of the round are issued before any is combined, so a
    // wave keeps 16 LDS reads in flight
    const uint32_t a0 = GIFT_T0(s0, 0), a1 = GIFT_T1(s1, 1), a2 = GIFT_T2(s2, 2), a3 = GIFT_T3(s3, 3);
    const uint32_t b0 = GIFT_T0(s1, 0), b1 = GIFT_T1(s2, 1), b2 = GIFT_T2(s3, 2), b3 = GIFT_T3(s0, 3);
    const uint32_t c0 = GIFT_T0(s2, 0), c1 = GIFT_T1(s3, 1), c2 = GIFT_T2(s0, 2), c3 = GIFT_T3(s1, 3);
    const uint32_t d0 = GIFT_T0(s3, 0), d1 = GIFT_T1(s0, 1), d2 = GIFT_T2(s1, 2), d3 = GIFT_T3(s2, 3);
    __builtin_amdgcn_sched_group_barrier(0x0002, 16, 0);  // 16 address perms
    __builtin_amdgcn_sched_group_barrier(0x0100, 16, 0);  // 16 LDS reads
    __builtin_amdgcn_sched_group_barrier(0x0002, 8, 0);   // 8 xor3
    __builtin_amdgcn_s_setprio(0);
    s0 = xor3(xor3(a0, a1, a2), a3, rk[4 * r + 0]);
    s1 = xor3(xor3(b0, b1, b2), b3, rk[4 * r + 1]);
    s2 = xor3(xor3(c0, c1, c2), c3, rk[4 * r + 2]);
    s3 = xor3(xor3(d0, d1, d2), d3, rk[4 * r + 3]);
  }
  // Last round: S(x) is byte 0 of T2[x], byte 1 of T3[x], byte 2 of T0[x],
  // byte 3 of T1[x]; v_perm merges them, and the halves do not overlap so
  // OR = XOR.
#define GIFT_LAST(a, b, c, d, rkw)                                                              \
  xor3(__builtin_amdgcn_perm(GIFT_T3(b, 1), GIFT_T2(a, 0), 0x0c0c0500u),                        \
       __builtin_amdgcn_perm(GIFT_T1(d, 3), GIFT_T0(c, 2), 0x07020c0cu), (rkw))
  const uint32_t o0 = GIFT_LAST(s0, s1, s2, s3, rk[56]);
  const uint32_t o1 = GIFT_LAST(s1, s2, s3, s0, rk[57]);
  const uint32_t o2 = GIFT_LAST(s2, s3, s0, s1, rk[58]);
  const uint32_t o3 = GIFT_LAST(s3, s0, s1, s2, rk[59]);
#undef GIFT_LAST
  s0 = o0;
  s1 = o1;
  s2 = o2;
  s3 = o3;
}

// Counter-mode caching of rounds 1-2.  In a tile, lane l encrypts the counter
// blocks IV || BE32(c + kThreads*r) for rows r, so (kThreads >= 256) the
// counter's low 8 bits never change for the lane; the first three state columns are the IV (uniform).
// After round 1 only column 1 depends on counter bits 8..15 (one lookup per
// row); columns 2 and 3 depend on bits 16..31, which change at most twice per
// tile; column 0 is fixed.  Round 2 then has one varying lookup per column.
// So per row rounds 1-2 cost 5 lookups instead of 32.
struct CtrCache {
  uint32_t u1, u2, u3, in0;  // round-1 partial columns
  uint32_t in2, in3;         // round-1 columns 2, 3 for the current counter bits 16..31
  uint32_t w0, w1, w2, w3;   // round-2 partial columns
  uint32_t hi;               // counter bits 16..31 the cache was built for
};

__device__ __forceinline__ void ctr_cache_init(CtrCache& c, uint32_t k0, uint32_t k1, uint32_t k2, uint32_t c0,
                                               const uint32_t* rk, const uint8_t* tt, uint32_t L) {
  // every lane reads its own table copy, so these are equal across the wave
  const uint32_t u0 = __builtin_amdgcn_readfirstlane(xor3(GIFT_T0(k0, 0), GIFT_T1(k1, 1), GIFT_T2(k2, 2)) ^ rk[4]);
  c.u1 = __builtin_amdgcn_readfirstlane(xor3(GIFT_T0(k1, 0), GIFT_T1(k2, 1), GIFT_T3(k0, 3)) ^ rk[5]);
  c.u2 = __builtin_amdgcn_readfirstlane(xor3(GIFT_T0(k2, 0), GIFT_T2(k0, 2), GIFT_T3(k1, 3)) ^ rk[6]);
  c.u3 = __builtin_amdgcn_readfirstlane(xor3(GIFT_T1(k0, 1), GIFT_T2(k1, 2), GIFT_T3(k2, 3)) ^ rk[7]);
  c.in0 = u0 ^ GIFT_T3(bswap32(c0) ^ rk[3], 3);  // counter byte 15: fixed per lane
  c.hi = ~(c0 >> 16);                            // forces a refresh on first use
}

// Round-2 output for counter ctr (state after rounds 1 and 2).
__device__ __forceinline__ void ctr_rounds12(CtrCache& c, uint32_t ctr, uint32_t& x0, uint32_t& x1, uint32_t& x2,
                                             uint32_t& x3, const uint32_t* rk, const uint8_t* tt, uint32_t L) {
  const uint32_t s3 = bswap32(ctr) ^ rk[3];
  if ((ctr >> 16) != c.hi) {  // rare and per lane
    c.hi = ctr >> 16;
    const uint32_t in0 = opaque(c.in0);  // its lookups stay here, not held in registers across the rows
    c.in2 = c.u2 ^ GIFT_T1(s3, 1);
    c.in3 = c.u3 ^ GIFT_T0(s3, 0);
    c.w0 = xor3(GIFT_T0(in0, 0), GIFT_T2(c.in2, 2), GIFT_T3(c.in3, 3)) ^ rk[8];
    c.w1 = xor3(GIFT_T1(c.in2, 1), GIFT_T2(c.in3, 2), GIFT_T3(in0, 3)) ^ rk[9];
    c.w2 = xor3(GIFT_T0(c.in2, 0), GIFT_T1(c.in3, 1), GIFT_T2(in0, 2)) ^ rk[10];
    c.w3 = xor3(GIFT_T0(c.in3, 0), GIFT_T1(in0, 1), GIFT_T3(c.in2, 3)) ^ rk[11];
  }
  const uint32_t in1 = c.u1 ^ GIFT_T2(s3, 2);
  x0 = c.w0 ^ GIFT_T1(in1, 1);
  x1 = c.w1 ^ GIFT_T0(in1, 0);
  x2 = c.w2 ^ GIFT_T3(in1, 3);
  x3 = c.w3 ^ GIFT_T2(in1, 2);
}

// Y*M xor X with the 32 nibble tables of M in LDS: nibble q of Y (GCM bits
// 4q..4q+3; q even = high nibble of byte q/2) selects entry q*256 + v*16.
// 16 * (high nibble of byte k of w) and 16 * (low nibble of byte k of w),
// one SDWA instruction each (byte select on the source; for the low nibble
// the shifted byte is written to byte 0 of a zeroed result).
__device__ __forceinline__ uint32_t nib_hi16(uint32_t w, int k) {
  uint32_t r;
  switch (k) {
    case 0: asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD" : "=v"(r) : "v"(w), "v"(0xF0u)); break;
    case 1: asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD" : "=v"(r) : "v"(w), "v"(0xF0u)); break;
    case 2: asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD" : "=v"(r) : "v"(w), "v"(0xF0u)); break;
    default: asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD" : "=v"(r) : "v"(w), "v"(0xF0u)); break;
  }
  return r;
}
__device__ __forceinline__ uint32_t nib_lo16(uint32_t w, int k) {
  uint32_t r;
  switch (k) {
    case 0: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(4u), "v"(w)); break;
    case 1: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(4u), "v"(w)); break;
    case 2: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(4u), "v"(w)); break;
    default: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(4u), "v"(w)); break;
  }
  return r;
}

__device__ __forceinline__ u128 ghash_step_lds(const u128& y, const u128& x, const uint8_t* gt) {
  uint32_t a0 = x.w[0], a1 = x.w[1], a2 = x.w[2], a3 = x.w[3];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    // eight table reads per word of Y in flight, then an xor tree
    const uint32_t w = y.w[j];
    uint4 e[8];
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int q = 2 * (4 * j + k);
      e[2 * k] = lds128(gt + q * 256, nib_hi16(w, k));
      e[2 * k + 1] = lds128(gt + (q + 1) * 256, nib_lo16(w, k));
    }
    __builtin_amdgcn_sched_group_barrier(0x0002, 8, 1);  // addresses
    __builtin_amdgcn_sched_group_barrier(0x0100, 8, 1);  // 8 LDS reads
    __builtin_amdgcn_sched_group_barrier(0x0002, 16, 1); // xor3s
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
      a0 = xor3(a0, e[k].x, e[k + 1].x);
      a1 = xor3(a1, e[k].y, e[k + 1].y);
      a2 = xor3(a2, e[k].z, e[k + 1].z);
      a3 = xor3(a3, e[k].w, e[k + 1].w);
    }
  }
  return u128{{a0, a1, a2, a3}};
}

// The first n (1..16) bytes of a block at any address.  Global loads and
// stores of any width may be unaligned on gfx950, so a whole block is one
// 16-byte access and a partial one up to four (8, 4, 2, 1 bytes).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef uint64_t u64_any __attribute__((aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
__device__ __forceinline__ u128 load_block(const uint8_t* p, uint32_t n) {
  if (n == 16) {
    const u32x4 v = *(const u32x4_any*)p;
    return u128{{v.x, v.y, v.z, v.w}};
  }
  const uint32_t hi = n & 8u;
  uint64_t v = 0;
  uint32_t w = 0, t = 0;  // the 4 bytes after those (or at the start), then the last up to 3
  if (hi) v = *(const u64_any*)p;
  if (n & 4u) w = *(const u32_any*)(p + hi);
  if (n & 2u) t = *(const u16_any*)(p + (n & 12u));
  if (n & 1u) t |= (uint32_t)p[n & 14u] << (8u * (n & 2u));
  const uint32_t a = (n & 4u) ? w : t, b = (n & 4u) ? t : 0u;
  return u128{{hi ? (uint32_t)v : a, hi ? (uint32_t)(v >> 32) : b, hi ? a : 0u, hi ? b : 0u}};
}

__device__ __forceinline__ void store_block(uint8_t* p, const u128& v, uint32_t n) {
  if (n == 16) {
    *(u32x4_any*)p = u32x4{v.w[0], v.w[1], v.w[2], v.w[3]};
    return;
  }
  const uint32_t v0 = v.w[0], v1 = v.w[1], v2 = v.w[2], v3 = v.w[3];
  const uint32_t hi = n & 8u, w = hi ? v2 : v0, w1 = hi ? v3 : v1;
  const uint32_t t = (n & 4u) ? w1 : w;
  if (hi) *(u64_any*)p = ((uint64_t)v1 << 32) | v0;
  if (n & 4u) *(u32_any*)(p + hi) = w;
  if (n & 2u) *(u16_any*)(p + (n & 12u)) = (uint16_t)t;
  if (n & 1u) p[n & 14u] = (uint8_t)(t >> (8u * (n & 2u)));
}

// keep the first n bytes of a block, zero the rest
__device__ __forceinline__ u128 mask_block(const u128& v, uint32_t n) {
  if (n >= 16) return v;
  u128 r = v;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    int keep = (int)n - 4 * j;
    uint32_t m = keep >= 4 ? 0xFFFFFFFFu : (keep <= 0 ? 0u : ((1u << (8 * keep)) - 1u));
    r.w[j] &= m;
  }
  return r;
}

// Whole-block stream of the per-block kernel: every plaintext and ciphertext
// block passes through the caches once, so its 16-byte load and store carry
// the non-temporal hint.  Measured on llama3_8b_kv: seal kernel -0.75%.
__device__ __forceinline__ uint4 ld_stream(const uint8_t* p) {
  const u32x4 t = __builtin_nontemporal_load((const u32x4_any*)p);
  return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st_stream(uint8_t* p, const uint4& v) {
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, (u32x4_any*)p);
}

__device__ __forceinline__ u128 ld_u128(const uint4* p) {
  uint4 v = *p;
  return u128{{v.x, v.y, v.z, v.w}};
}
__device__ __forceinline__ void st_u128(uint4* p, const u128& v) { *p = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]); }

// GHASH length block 0^64 || BE64(8*len) as block words.
__device__ __forceinline__ u128 length_block(uint64_t len) {
  uint64_t bits = len * 8ull;
  return u128{{0u, 0u, bswap32((uint32_t)(bits >> 32)), bswap32((uint32_t)bits)}};
}

// A wave's share of a tile's sum: each lane's y times the lane's power hp,
// summed over the wave (the result is wave-uniform).  Kept out of line, so
// that the main loop's register allocation does not see the multiply
// (inlined, the kernel spills).
__device__ __noinline__ u128 wave_sum_of(u128 y, u128 hp) {
  u128 z = gf_mul(y, hp);
#pragma unroll
  for (int j = 0; j < 4; j++) z.w[j] = wave_xor(z.w[j]);
  return z;
}

// The lane's index (the thread index would be an argument of an out-of-line
// function, held in a register throughout its caller).
__device__ __forceinline__ uint32_t lane_index() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
// Global memory as such, for out-of-line functions (through generic pointers
// their accesses would be flat ones).
typedef const __attribute__((address_space(1))) u32x4* global_block;
typedef const __attribute__((address_space(1))) uint32_t* global_word;
__device__ __forceinline__ u128 ld_global(global_block p) {
  const u32x4 v = *p;
  return u128{{v.x, v.y, v.z, v.w}};
}
// gf_mul_wave out of line, for the same reason as wave_sum_of.
__device__ __noinline__ u128 wave_mul(u128 x, u128 y) { return gf_mul_wave(x, y, lane_index()); }

// What the tag of a segment needs besides its blocks: E_K(J0) xor H*L, J0 = IV
// || BE32(1), by one wave (the result is wave-uniform).  r and tt: the segment's
// TileInfo and the T-tables; H*L is a wave sum over the set bits of the length
// block (only its low 64 bits can be set) of the products hxl = H * x^(64+k).
// Out of line, as wave_sum_of; LDS comes as LDS pointers, not generic ones.
typedef const __attribute__((address_space(3))) uint32_t* lds_words;
__device__ __noinline__ u128 tag_mask(lds_words r, lds_words tt, global_block hxl) {
  const uint32_t lane = lane_index();
  auto word = [&](size_t at) { return (uint32_t)__builtin_amdgcn_readfirstlane(r[at / 4]); };
  const uint64_t len = (uint64_t)word(offsetof(TileInfo, desc) + offsetof(SegDesc, len) + 4) << 32 |
                       word(offsetof(TileInfo, desc) + offsetof(SegDesc, len));
  u128 z = u128_zero();
  if (((len * 8ull) >> (63 - lane)) & 1ull) z = ld_global(hxl + lane);
  constexpr size_t iv = offsetof(TileInfo, desc) + offsetof(SegDesc, iv), rk = offsetof(TileInfo, rk);
  uint32_t s0 = word(iv) ^ word(rk), s1 = word(iv + 4) ^ word(rk + 4), s2 = word(iv + 8) ^ word(rk + 8),
           s3 = 0x01000000u ^ word(rk + 12);
  // table k of byte k, this lane's copy
  const lds_words c = tt + (lane & 31u);
  auto te = [&](uint32_t w, uint32_t k) -> uint32_t {
    return c[(((w >> (8u * k)) & 0xFFu) << 6) + 32u * (k & 1u) + 16384u * (k >> 1)];
  };
#pragma unroll 1
  for (uint32_t i = 1; i < 14u; i++) {
    const lds_words k = r + rk / 4 + 4u * i;
    const uint32_t t0 = xor3(te(s0, 0), te(s1, 1), te(s2, 2)) ^ te(s3, 3) ^ k[0];
    const uint32_t t1 = xor3(te(s1, 0), te(s2, 1), te(s3, 2)) ^ te(s0, 3) ^ k[1];
    const uint32_t t2 = xor3(te(s2, 0), te(s3, 1), te(s0, 2)) ^ te(s1, 3) ^ k[2];
    const uint32_t t3 = xor3(te(s3, 0), te(s0, 1), te(s1, 2)) ^ te(s2, 3) ^ k[3];
    s0 = t0, s1 = t1, s2 = t2, s3 = t3;
  }
  // S(x) is byte 1 of T0[x] (bytes 2S, S, S, 3S)
  auto sb = [&](uint32_t w, uint32_t k) -> uint32_t {
    const uint32_t x = c[((w >> (8u * k)) & 0xFFu) << 6];
    return ((x >> 8) & 0xFFu) << (8u * k);
  };
  const uint32_t o[4] = {sb(s0, 0) | sb(s1, 1) | sb(s2, 2) | sb(s3, 3), sb(s1, 0) | sb(s2, 1) | sb(s3, 2) | sb(s0, 3),
                         sb(s2, 0) | sb(s3, 1) | sb(s0, 2) | sb(s1, 3), sb(s3, 0) | sb(s0, 1) | sb(s1, 2) | sb(s2, 3)};
#pragma unroll
  for (int j = 0; j < 4; j++) z.w[j] = wave_xor(z.w[j]) ^ __builtin_amdgcn_readfirstlane(o[j]) ^ word(rk + 4 * (56 + j));
  return z;
}

// Tiles of a segment of m blocks.
__device__ __forceinline__ uint32_t tiles_in(uint32_t nblocks) {
  return (uint32_t)(((uint64_t)nblocks + kTileBlocks - 1) / kTileBlocks);
}

// Rows of tile t of a segment of m blocks (tiles aligned to its end: only the
// first tile, t = tiles - 1, can be partial).
__device__ __forceinline__ uint32_t tile_rows_of(uint32_t m, uint32_t t) {
  const int64_t base = (int64_t)m - (int64_t)(t + 1) * (int64_t)kTileBlocks;
  return base >= 0 ? (uint32_t)kRows : (uint32_t)kRows - (uint32_t)((uint64_t)(-base) / kThreads);
}

// sum_t P_t H^(tT) over the nt tile partials of a segment, by one wave: lane l
// folds tiles l, l + 64, ...; with up to four tiles, 16 lanes share a tile's
// product.  ht: H^(lT) of lane l; hlt: H^(64T).  The partials were written by
// other workgroups of this launch, so they are read past the caches.
//
// It runs in the tile kernel, by the wave that completes the segment.  As a
// kernel of its own behind the tile kernel it took 4.0 us for one segment of 8
// tiles, nearly all of it the launch.
__device__ __noinline__ u128 fold_tiles(global_word partials, uint32_t nt, global_block ht, global_block hlt) {
  const uint32_t lane = lane_index();
  auto part = [&](uint32_t t) -> u128 {
    u128 v;
#pragma unroll
    for (int j = 0; j < 4; j++)
      v.w[j] = __hip_atomic_load(partials + 4ull * t + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return v;
  };
  u128 z = u128_zero();
  if (nt <= 4u) {
    const uint32_t t = lane >> 4;
    if (t < nt) {
      const u128 x = part(t);
      if (t > 0u)
        z = gf_mul_slice(x, ld_global(ht + t), lane & 15u);
      else if (lane == 0u)
        z = x;
    }
  } else if (lane < nt) {
    const uint32_t K = (nt - 1 - lane) / kFinLanes + 1;
    const u128 hl = ld_global(ht + lane);
    z = part(lane + (K - 1) * kFinLanes);
    if (K > 1) {
      const u128 h64 = ld_global(hlt);
      for (int k = (int)K - 2; k >= 0; k--) z = u128_xor(gf_mul(z, h64), part(lane + (uint32_t)k * kFinLanes));
    }
    if (lane > 0) z = gf_mul(z, hl);
  }
#pragma unroll
  for (int j = 0; j < 4; j++) z.w[j] = wave_xor(z.w[j]);
  return z;
}

// Zeroes len bytes (at most a tile's) at any address, by one wave.  The other
// waves of the team are in the next tile, so the wave has to keep as many
// stores under way as it can: whole blocks without a look at the segment's end.
// Opens in which every tag fails, block by block with that look / so: 300
// segments of 0.5 MiB 344 / 296 us per call, 256 of them 192 / 165, 600 of 2 MiB
// 1826 / 1680.
typedef __attribute__((address_space(1))) uint8_t* global_bytes;
__device__ __noinline__ void zero_tile(global_bytes p, uint32_t len) {
  typedef __attribute__((address_space(1))) u32x4_any* blocks;
  const uint32_t lane = lane_index(), whole = len / 16u;
  const blocks q = (blocks)p + lane;
  uint32_t i = 0;
  for (; i + 512u <= whole; i += 512u)
#pragma unroll
    for (uint32_t k = 0; k < 512u; k += 64u) q[i + k] = u32x4{0u, 0u, 0u, 0u};
  for (; i + lane < whole; i += 64u) q[i] = u32x4{0u, 0u, 0u, 0u};
  if (lane < (len & 15u)) p[16u * whole + lane] = 0;
}

// ---------------------------------------------------------------------------
// Per-block kernel over 2 MiB tiles of the non-small segments.
// ---------------------------------------------------------------------------
template <int MODE, int TEAMS>
__global__ __launch_bounds__(kThreads) void k_gcm_tiles(GcmArgs a) {
  constexpr uint32_t kTeamThreads = Team<TEAMS>::threads, kTeamWaves = Team<TEAMS>::waves;
  constexpr int kTeamRows = Team<TEAMS>::rows;
  constexpr bool OPEN = (MODE & kModeOpen) != 0;
  constexpr bool GATHER = (MODE & kModeGather) != 0, SCATTER = (MODE & kModeScatter) != 0;
  __shared__ __attribute__((aligned(16))) uint8_t smem[Team<TEAMS>::lds_bytes];
  const uint32_t tid = threadIdx.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t team = wave / kTeamWaves, tw = wave % kTeamWaves;
  uint8_t* tt = smem + Team<TEAMS>::lds_aes;
  TeamState* const ts = (TeamState*)(smem + Team<TEAMS>::lds_state) + team;

  // The record of queue entry i, by one wave (lane l of it).
  auto load_record = [&](TileInfo* t, uint32_t i, uint32_t l) {
    const TileEnt e = i < a.n_ents ? a.tile_order[i] : TileEnt{kNoTile, 0u, 0u, 0u};
    if (l == 0u) *(uint4*)t = make_uint4(e.g, e.s, e.trow, e.user);
    if (e.g == kNoTile) return;
    t->rk[l] = a.kt.rk[(size_t)e.user * 64u + l];
    if (l < 16u) ((uint32_t*)&t->desc)[l] = ((const uint32_t*)(a.segs + e.s))[l];
    if (l == 16u) t->verdict = a.verdicts[e.s];
  };
  // the tables of M of a user, by one wave: two calls, so that the loads can
  // be in flight while the team finishes with the tables before them
  struct Tables {
    u32x4 e0, e1, e2, e3, e4, e5, e6, e7;
  };
  auto read_tables = [&](uint32_t user, uint32_t l) -> Tables {
    const u32x4* src = (const u32x4*)(a.kt.gtab + ((size_t)user * 2u + (TEAMS - 1u)) * 512u) + l;
    return Tables{src[0], src[64], src[128], src[192], src[256], src[320], src[384], src[448]};
  };
  auto write_tables = [&](const Tables& m, uint32_t l) {
    u32x4* dst = (u32x4*)(smem + team * kGtabBytes) + l;
    dst[0] = m.e0, dst[64] = m.e1, dst[128] = m.e2, dst[192] = m.e3;
    dst[256] = m.e4, dst[320] = m.e5, dst[384] = m.e6, dst[448] = m.e7;
  };

  // Work queue over the expansion's order (longest entries first): team w of
  // W takes entry w first, then entries W + (queue claims).  Two teams per
  // workgroup run short tiles, most often two each: there the second entry is
  // 2W - 1 - w (the longest with the shortest), known at the start.
  //
  // The waves of a team go through its tiles without a barrier, each at its
  // own pace, so that one tile's end (the generic multiplies, VALU work of
  // about 900 instructions per wave) overlaps LDS work of the other waves:
  //   - kRecWave, of the oldest waves, which the SIMDs favour and which finish
  //     first, fetches tile k + 1's record (queue claim, entry, descriptor and
  //     round keys: three dependent loads, up to 12k clocks).  In a tile of
  //     more than kLateRows rows it does so after its rows, so that a
  //     workgroup claims no more than it is about to run; else before them.
  //     Early in every tile of up to 16 rows, a workgroup that came from a
  //     longer one claimed two short entries at once, and others went without:
  //     seals of 256 segments of 48 rows (32-row pieces, then 16) 286 us per
  //     call, late from 3 rows on 223; 531 segments of 1-60 rows 352 / 304, 795
  //     of them 511 / 463; in tiles of 1-4 rows no difference.
  //     The slot held tile k - 3, which is finished.
  //   - a wave that has done its rows of tile k multiplies, adds to the tile's
  //     sum and goes on to tile k + 1, whose first row needs no GHASH table.
  //   - kTabWave, of the youngest, writes the tables of tile k + 1's user once
  //     every wave of the team has done its rows of tile k.
  //   - the last wave to add its sum finishes the tile.
  // Against barriers around the tile's end and four leader waves folding all
  // partials there (per-phase clocks: LDS idle for 46% of the time with 1-4
  // rows per tile): 1024 segments of 16-64 KiB 80.4 -> 74.0 us per call with
  // two teams (81 with one); 2 requests, 45 tiles cut into 25-row pieces, 159.9
  // -> 144.2 us; 128-row tiles +0.7%.
  constexpr uint32_t kRecWave = 0, kTabWave = kTeamWaves - 1;
  constexpr int kLateRows = 2 * TEAMS;  // 2 rows of 1024 blocks
  constexpr bool kPair = TEAMS == 2;  // the second entry is 2W - 1 - w
  const uint32_t W = TEAMS * gridDim.x, w = blockIdx.x + team * gridDim.x;
  const TileEnt e0 = w < a.n_ents ? a.tile_order[w] : TileEnt{kNoTile, 0u, 0u, 0u};

  // Replicated T-tables: word w = region*16384 + x*64 + slot holds
  // T_{2*region + slot/32}[x] = rotl(Te0[x], 8*table).  Four consecutive
  // slots hold the same word, so each thread writes 16 bytes at a time.
  for (uint32_t q = tid; q < 8192u; q += kThreads) {
    const uint32_t w = 4u * q;
    const uint32_t region = w >> 14, x = (w >> 6) & 255u, slot = w & 63u;
    const uint32_t tab = 2u * region + (slot >> 5);
    const uint32_t v = c_aes.te0[x];
    const uint32_t sh = 8u * tab;
    const uint32_t r = (v << sh) | (v >> ((32u - sh) & 31u));
    ((uint4*)tt)[q] = make_uint4(r, r, r, r);
  }
  const uint32_t L = ((tid & 31u) << 2) | 0x10000u;  // this lane's table copy
  // the first tile's tables, the first two records
  if (tw == kTabWave && e0.g != kNoTile) write_tables(read_tables(e0.user, tid & 63u), tid & 63u);
  if (tw == kRecWave) load_record(&ts->info[0], w, tid & 63u);
  if (kPair && tw == 1) load_record(&ts->info[1], 2u * W - 1u - w, tid & 63u);
  if (tw == 2) {
    if ((tid & 63u) < kSlots) ts->sum[tid & 63u] = TileSum{{0u, 0u, 0u, 0u}, 0u, 0u, {0u, 0u}};
    if ((tid & 63u) == 0u) ts->rec = kPair ? 2u : 1u, ts->mtab = 1u, ts->fin = 0u;
  }
  __syncthreads();

  auto fetch_next = [&](uint32_t k, uint32_t l) {
    if (kPair && k == 0u) return;
    uint32_t c = 0;
    if (l == 0u) c = atomicAdd(a.tile_counter, 1u);
    c = (uint32_t)__builtin_amdgcn_readfirstlane(c) + (kPair ? 2u * W : W);
    wave_wait(&ts->fin, k - 2u);
    load_record(&ts->info[(k + 1u) % kSlots], c, l);
    wave_set(&ts->rec, k + 2u);
  };
  for (uint32_t k = 0;; k++) {
    wave_wait(&ts->rec, k + 1u);
    const TileInfo* ti = &ts->info[k % kSlots];
    if ((uint32_t)__builtin_amdgcn_readfirstlane(ti->g) == kNoTile) break;
    // the thread index, recomputed per tile: per-lane values derived from it
    // are formed here, not hoisted to the kernel's start and held (or
    // spilled) across every tile
    const uint32_t tid_t = opaque(tid) % kTeamThreads;
    const uint32_t trow = __builtin_amdgcn_readfirstlane(ti->trow);
    const uint32_t t = trow & 0xFFFFu;                                      // tile of the segment
    // its rows in this entry, in the team's rows
    const int r0 = TEAMS * (int)((trow >> 16) & 0xFFu), r1 = TEAMS * (int)(trow >> 24);
    const uint32_t user = __builtin_amdgcn_readfirstlane(ti->user);
    const int32_t verdict = (int32_t)__builtin_amdgcn_readfirstlane((uint32_t)ti->verdict);
    const uint32_t m = __builtin_amdgcn_readfirstlane(ti->desc.nblocks);
    const uint64_t off = uniform64(ti->desc.byte_off), len = uniform64(ti->desc.len);
    const int64_t base = (int64_t)m - (int64_t)(t + 1) * (int64_t)kTileBlocks;  // block index of virtual slot 0
    const int r_start = base < 0 ? (int)((uint64_t)(-base) / kTeamThreads) : 0;
    const int r_lo = r_start > r0 ? r_start : r0;
    const bool late = r1 - r_lo > kLateRows;
    if (tw == kRecWave && !late) fetch_next(k, tid_t & 63u);

    // paged side: block i of the segment lives in chunk i >> shift
    const uint64_t chunk0 = uniform64(ti->desc.chunk0);
    const uint64_t cmask = (1ull << a.chunk_shift) - 1;
    auto paged = [&](uint64_t i) -> uint8_t* {
      return a.pbase + a.chunk_off[chunk0 + (i >> a.chunk_shift)] + ((i & cmask) << 4);
    };

    // Tile-uniform values are read from the tile record into SGPRs
    // (readfirstlane), so the per-block loop keeps no copy of the 60
    // round-key words in VGPRs.
    uint32_t rk[60];
#pragma unroll
    for (int i = 0; i < 60; i++) rk[i] = __builtin_amdgcn_readfirstlane(ti->rk[i]);
    const uint32_t k0 = __builtin_amdgcn_readfirstlane(ti->desc.iv[0]) ^ rk[0];
    const uint32_t k1 = __builtin_amdgcn_readfirstlane(ti->desc.iv[1]) ^ rk[1];
    const uint32_t k2 = __builtin_amdgcn_readfirstlane(ti->desc.iv[2]) ^ rk[2];

    u128 y = u128_zero();
    if (verdict != kVerdictOk) {
      // rejected before this call's data is touched: release zeros only.  A
      // scatter into the cache writes nothing at all: the request's table
      // names a block of another owner, which keeps its contents.
      if (!SCATTER) {
        const uint32_t z = opaque(0u);  // formed here, not held from the kernel's start
        for (int r = r_lo; r < r1; r++) {
          const int64_t i0 = base + (int64_t)r * kTeamThreads + tid_t;
          if (i0 >= 0) {
            const uint64_t rem = len - 16ull * (uint64_t)i0;
            store_block(a.out + off + 16ull * (uint64_t)i0, u128{{z, z, z, z}}, rem >= 16 ? 16u : (uint32_t)rem);
          }
        }
      }
    } else {
      CtrCache cc;
      const uint32_t c0 = 2u + (uint32_t)(base + (int64_t)tid_t);  // counter of this lane in row 0, mod 2^32
      ctr_cache_init(cc, k0, k1, k2, c0, rk, tt, L);

      // Rows where every lane holds a whole block take the branch-free path,
      // whatever the segment's alignment (256 prompts of int32 tokens, most of
      // them unaligned: kernel 27.8 -> 21.9 us against byte loads and stores).
      const int r_full = base < 0 ? (int)(((uint64_t)(-base) + kTeamThreads - 1) / kTeamThreads) : 0;
      const int r_end_full = (t == 0 && (len & 15u)) ? r1 - (r1 == kTeamRows ? 1 : 0) : r1;

      auto whole = [&](int r) { return r >= r_full && r < r_end_full; };
      // paged: a lane's chunk offset for the next whole-block row is loaded
      // one row ahead, so the gather or scatter address is ready when the row
      // starts
      constexpr bool PAGED = GATHER || SCATTER;
      auto chunk_of = [&](int r) -> uint64_t {
        const uint64_t i0 = (uint64_t)(base + (int64_t)r * kTeamThreads + tid_t);
        return a.chunk_off[chunk0 + (i0 >> a.chunk_shift)];
      };
      uint64_t c_next = (PAGED && whole(r_lo)) ? chunk_of(r_lo) : 0;

      for (int r = r_lo; r < r1; r++) {
        // the whole-block rows load their input before the AES rounds, so the
        // HBM latency overlaps the keystream
        const bool fast = whole(r);
        const uint64_t c_cur = c_next;
        if (PAGED && whole(r + 1)) c_next = chunk_of(r + 1);
        const uint8_t* src = nullptr;
        uint8_t* dst = nullptr;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (fast) {
          // every lane's block index is >= 0 in these rows; pointer arithmetic
          // (not integers) keeps the global address space for the compiler
          const uint64_t i0 = (uint64_t)(base + (int64_t)r * kTeamThreads + tid_t);
          uint8_t* pg = a.pbase + c_cur + ((i0 & cmask) << 4);
          src = GATHER ? pg : a.in + off + 16ull * i0;
          dst = SCATTER ? pg : a.out + off + 16ull * i0;
          v = ld_stream(src);
        }
        uint32_t x0, x1, x2, x3;
        ctr_rounds12(cc, c0 + (uint32_t)kTeamThreads * (uint32_t)r, x0, x1, x2, x3, rk, tt, L);
        aes_rounds_lds<3>(x0, x1, x2, x3, rk, tt, L);
        u128 x;
        if (fast) {
          const uint4 o = make_uint4(v.x ^ x0, v.y ^ x1, v.z ^ x2, v.w ^ x3);
          st_stream(dst, o);
          x = OPEN ? u128{{v.x, v.y, v.z, v.w}} : u128{{o.x, o.y, o.z, o.w}};
        } else {
          x = u128_zero();
          const int64_t i0 = base + (int64_t)r * kTeamThreads + tid_t;
          if (i0 >= 0) {
            const uint64_t boff = off + 16ull * (uint64_t)i0;
            const uint64_t rem = len - 16ull * (uint64_t)i0;
            const uint32_t n = rem >= 16 ? 16u : (uint32_t)rem;
            const u128 in = load_block(GATHER ? paged((uint64_t)i0) : a.in + boff, n);
            const u128 o = mask_block(u128{{in.w[0] ^ x0, in.w[1] ^ x1, in.w[2] ^ x2, in.w[3] ^ x3}}, n);
            store_block(SCATTER ? paged((uint64_t)i0) : a.out + boff, o, n);
            x = OPEN ? in : o;
          }
        }
        // The first row's running sum is zero: nothing to multiply.  With 1-4
        // KiB rows per tile (1024 segments of 16-64 KiB) a seal call went from
        // 84.2 to 80.4 us; tiles of 128 rows do not notice.
        if (r == r_lo) {
          y = x;
          if (r + 1 < r1) wave_wait(&ts->mtab, k + 1u);
        } else {
          // GHASH table reads at a priority between the AES issue and combine
          // phases; the next AES round sets its own.  One copy per team: the
          // tables' place goes into the reads' immediate offsets.
          __builtin_amdgcn_s_setprio(1);
          if (TEAMS == 1 || team == 0u)
            y = ghash_step_lds(y, x, smem);
          else
            y = ghash_step_lds(y, x, smem + kGtabBytes);
        }
      }
    }  // verdict OK

    // Tile end: lane tid_t contributes y * H^(kTeamThreads + 1 - tid_t), its
    // distance from the tile end plus the H^2 that every block's GHASH term
    // carries.
    const bool fold = verdict == kVerdictOk;
    const uint32_t tid_e = opaque(tid) % kTeamThreads, lane = tid_e & 63u;
    TileSum* sum = &ts->sum[k % kSlots];
    if (tw == kRecWave && late) fetch_next(k, lane);
    u128 hp = u128_zero();
    if (fold) hp = ld_u128(a.kt.pow_h + (size_t)user * kHPowers + (kTeamThreads + 1u - tid_e));
    wave_wait(&ts->fin, k - (kSlots - 1u));  // the slot's previous tile is finished
    const bool first = wave_arrive(&sum->rows) == 0u;
    if (tw == kTabWave) {
      const TileInfo* tn = &ts->info[(k + 1u) % kSlots];
      wave_wait(&ts->rec, k + 2u);
      const uint32_t nu = __builtin_amdgcn_readfirstlane(tn->user);
      if ((uint32_t)__builtin_amdgcn_readfirstlane(tn->g) != kNoTile && nu != user) {
        const Tables m = read_tables(nu, lane);
        wave_wait(&sum->rows, kTeamWaves);
        write_tables(m, lane);
      }
      wave_set(&ts->mtab, k + 2u);
    }
    if (fold) {
      u128 z = wave_sum_of(y, hp);
      // The rest of the tag, by the first wave that is through the rows of the
      // segment's end, whose sum no power of H multiplies any more.  The other
      // waves are still in their rows.  In the prologue, where a wave per
      // segment formed it from tables of its own, it was the longest part: one
      // 16 MiB segment 7.7 us, without it 4; 1024 segments 10.8 and 6.
      if (first && t == 0u && r1 == kTeamRows)
        z = u128_xor(z, tag_mask((lds_words)(const uint32_t*)ti, (lds_words)(const uint32_t*)tt,
                                 (global_block)(a.kt.pow_hxl + (size_t)user * kHxLanes)));
      if (lane < 4u)
        atomicXor(&sum->z[lane], lane == 0u ? z.w[0] : lane == 1u ? z.w[1] : lane == 2u ? z.w[2] : z.w[3]);
    }
    if (wave_arrive(&sum->done) != kTeamWaves - 1u) continue;

    // The last wave of the team finishes the tile; lane 0 writes.  What only
    // this part needs of the record is read here, not held across the rows.
    const uint32_t g = __builtin_amdgcn_readfirstlane(ti->g), s = __builtin_amdgcn_readfirstlane(ti->s);
    const uint32_t m_e = __builtin_amdgcn_readfirstlane(ti->desc.nblocks);
    const uint32_t trow_e = __builtin_amdgcn_readfirstlane(ti->trow), t_e = trow_e & 0xFFFFu;
    const uint32_t p0 = (trow_e >> 16) & 0xFFu, p1 = trow_e >> 24;  // its rows, of kThreads blocks
    const uint32_t flags = __builtin_amdgcn_readfirstlane(ti->desc.flags);
    const uint32_t user_e = __builtin_amdgcn_readfirstlane(ti->user);
    const uint64_t off_e = uniform64(ti->desc.byte_off), len_e = uniform64(ti->desc.len);
    const bool one = (flags & kSegOneTile) != 0 && p0 == 0u && p1 == (uint32_t)kRows;  // the tile is the whole segment
    u128 p = u128{{sum->z[0], sum->z[1], sum->z[2], sum->z[3]}};
    if (lane < 8u) ((uint32_t*)sum)[lane] = 0u;  // the slot is free for tile k + kSlots
    wave_set(&ts->fin, k + 1u);
    if (!fold) {
      if (!OPEN && lane < 4u) ((uint32_t*)(a.tags_out + 16ull * s))[lane] = 0u;  // rejected: zero tag
      continue;
    }
    if (!one) {
      // A piece of a cut tile: its lane powers assumed rows up to the tile's
      // end, so it still carries H^(kThreads * (kRows - p1)); pieces
      // meet in the tile's (zeroed) partial by XOR.
      if (p1 < (uint32_t)kRows) p = wave_mul(p, ld_u128(a.kt.pow_hr + (size_t)user_e * kRows + (kRows - p1)));
      if (lane < 4u) {
        uint32_t* dst = (uint32_t*)(a.partials + g) + lane;
        const uint32_t v = lane == 0u ? p.w[0] : lane == 1u ? p.w[1] : lane == 2u ? p.w[2] : p.w[3];
        if (p0 == 0u && p1 == (uint32_t)kRows)
          __hip_atomic_store(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          __hip_atomic_fetch_xor(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // The entry that completes the segment's rows forms its tag.  The partials
      // are written and read by device-scope atomics, past the XCDs' caches, so
      // that the write above need only be complete before the rows count it.
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      const uint32_t nt = tiles_in(m_e), all = (nt - 1u) * kRows + tile_rows_of(m_e, nt - 1u);
      const uint32_t lo = kRows - tile_rows_of(m_e, t_e), mine = p1 - (p0 > lo ? p0 : lo);
      uint32_t before = 0;
      if (lane == 0u)
        before = __hip_atomic_fetch_add(a.seg_rows + s, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((uint32_t)__builtin_amdgcn_readfirstlane(before) + mine != all) continue;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      p = fold_tiles((global_word)(a.partials + (g - t_e)), nt, (global_block)(a.kt.pow_ht + (size_t)user_e * kFinLanes),
                     (global_block)(a.kt.pow_hlt + user_e));
    }
    // tag = E_K(J0) xor S, S = sum_t P_t H^(tT) xor H*L
    const u128 tag = p;
    if (!OPEN) {
      if (lane == 0) store_block(a.tags_out + 16ull * s, tag, 16u);
      continue;
    }
    const u128 want = load_block(a.tags_in + 16ull * s, 16u);
    uint32_t diff = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) diff |= want.w[j] ^ tag.w[j];
    const bool failed = __builtin_amdgcn_readfirstlane(diff) != 0;
    if (lane == 0) a.verdicts[s] = failed ? kVerdictAuthFail : kVerdictOk;
    if (!failed) continue;
    // Open of a contiguous tensor: a segment of one uncut tile whose tag failed
    // releases zeros only.  Its tile is the whole segment, so it is zeroed here,
    // after every wave's rows.  The others are zeroed by a later pass.
    if (SCATTER || !one) {
      if (lane == 0) *a.any_failed = 1u;
    } else {
      zero_tile((global_bytes)(a.out + off_e), (uint32_t)len_e);
    }
  }
}

// ---------------------------------------------------------------------------
// Segments of at most 64 blocks: one wave each.  Lane j < m owns block j and
// its GHASH term X_j * H^(m + 1 - j); lane m owns what is left of the tag, in
// the same steps: E_K(J0) instead of a keystream block (counter 1) and the
// length block's term L * H.  (With 64 blocks there is no lane m: lane 0 does
// that part in a second pass.)  Open decides the verdict before any plaintext
// is written.
//
// Bound by latency: dependent loads (list, descriptor, keys), 14 AES rounds,
// one generic product.  With E_K(J0) and L * H after the blocks instead of
// beside them, the product of up to four terms by one lane each instead of 16,
// and the round keys by vector loads inside the rounds, the kernel took 21.4 us
// for 1024 segments of 4 to 16 bytes; now 8.0 (a kernel that does nothing shows
// as 4).
// ---------------------------------------------------------------------------
template <bool OPEN>
__global__ __launch_bounds__(64) void k_small(GcmArgs a) {
  __shared__ uint32_t te[256];
  const uint32_t j = threadIdx.x;
  const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane(a.small_list[blockIdx.x]);
  const SegDesc sd = ld_uniform(a.segs + s);
  const uint32_t user = sd.user;
  const uint32_t rkv = a.kt.rk[(size_t)user * 64u + j];
  const uint32_t m = sd.nblocks;
  const bool valid = j < m, last = j == m;
  const uint64_t rem = valid ? sd.len - 16ull * j : 0;
  const uint32_t n = rem >= 16 ? 16u : (uint32_t)rem;
  uint8_t* dst = a.out + sd.byte_off + 16ull * j;
  const int32_t verdict = (int32_t)to_uniform((const uint32_t*)a.verdicts + s)[0];
  const u128 hp = j <= m ? ld_u128(a.kt.pow_h + (size_t)user * kHPowers + (m + 1 - j)) : u128_zero();
  u128 in = u128_zero();
  if (valid && verdict == kVerdictOk) in = load_block(a.in + sd.byte_off + 16ull * j, n);
  for (uint32_t i = j; i < 256u; i += 64u) te[i] = c_aes.te0[i];
  __syncthreads();
  if (verdict != kVerdictOk) {
    if (valid) store_block(dst, u128_zero(), n);
    if (!OPEN && j < 4) ((uint32_t*)(a.tags_out + 16ull * s))[j] = 0u;
    return;
  }
  const uint32_t cb[4] = {sd.iv[0], sd.iv[1], sd.iv[2], last ? 0x01000000u : bswap32(2u + j)};
  uint32_t ks[4];
  aes256_encrypt_tab(rkv, cb, ks, te);
  const u128 o = mask_block(u128{{in.w[0] ^ ks[0], in.w[1] ^ ks[1], in.w[2] ^ ks[2], in.w[3] ^ ks[3]}}, n);
  const u128 x = last ? length_block(sd.len) : OPEN ? in : o;
  u128 z;
  if (m < 4u) {
    // terms 0..m, 16 lanes each
    const uint32_t t = j >> 4;
    u128 tx = u128_zero(), th = u128_zero();
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int w = 0; w < 4; w++) {
        const uint32_t xw = (uint32_t)__builtin_amdgcn_readlane((int)x.w[w], i);
        const uint32_t hw = (uint32_t)__builtin_amdgcn_readlane((int)hp.w[w], i);
        if (t == (uint32_t)i) tx.w[w] = xw, th.w[w] = hw;
      }
    z = t <= m ? gf_mul_slice(tx, th, j & 15u) : u128_zero();
  } else {
    z = gf_mul(x, hp);  // hp is zero past the last term
  }
  if (m == 64u && j == 0u)
    z = u128_xor(z, gf_mul(length_block(sd.len), ld_u128(a.kt.pow_h + (size_t)user * kHPowers + 1)));
#pragma unroll
  for (int k = 0; k < 4; k++) z.w[k] = wave_xor(z.w[k]);
  // E_K(J0) xor the sum, wave-uniform
  u128 tag;
  if (m == 64u) {
    const uint32_t j0[4] = {sd.iv[0], sd.iv[1], sd.iv[2], 0x01000000u};
    aes256_encrypt_tab(rkv, j0, tag.w, te);
  } else {
#pragma unroll
    for (int k = 0; k < 4; k++) tag.w[k] = (uint32_t)__builtin_amdgcn_readlane((int)ks[k], (int)m);
  }
  tag = u128_xor(tag, z);
  bool ok = true;
  if (!OPEN) {
    if (j == 0u) store_block(a.tags_out + 16ull * s, tag, 16u);
  } else {
    const u128 want = load_block(a.tags_in + 16ull * s, 16u);
    uint32_t diff = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) diff |= want.w[k] ^ tag.w[k];
    ok = __builtin_amdgcn_readfirstlane(diff) == 0;
    if (j == 0u) a.verdicts[s] = ok ? kVerdictOk : kVerdictAuthFail;
  }
  if (valid) store_block(dst, ok ? o : u128_zero(), n);
}

// ---------------------------------------------------------------------------
// Segment-table expansion, by one workgroup of a call's first kernel: from
// the descriptors to the tables the GCM kernels read.
//   - tile_base: exclusive scan of the tiles of each segment (small segments
//     have none), tile_base[n] = all tiles;
//   - small_list: the small segments in table order;
//   - the cut: a tile runs on one CU, so with fewer tiles than CUs every
//     tile of more than p = ceil(all tile rows / CUs) rows is cut into
//     pieces of p rows; otherwise up to one tile per CU, the largest of more
//     than kPieceRows rows (in tile order within a row count), is cut into
//     pieces of kPieceRows rows.  Pieces are aligned to the tile's end; the
//     lowest may start below the tile's first row.  A one-tile segment
//     whose tile is cut is marked in seg_cut;
//   - the work queue: every whole tile and every piece, longest first (a
//     counting sort by the rows an entry runs), padded with kNoTile up to
//     cap entries.
// Each segment's tiles are split into runs of at most kRunTiles; threads
// take contiguous ranges of runs, so thread order is tile order.  Whole
// tiles and whole pieces take their slots by a scan over the threads, in
// tile order; the other entries (partial first tiles, remainder pieces) by
// LDS atomics, in no fixed order: which CU runs which entry changes no
// result.
// ---------------------------------------------------------------------------
constexpr int kExpandThreads = 1024;  // the most threads an expanding workgroup may have
constexpr int kPrologueThreads = kExpandThreads;  // the most; 256 for tables that fit them
// Waves of a workgroup that take a segment each: what its smallest workgroup
// has (with 16 in workgroups of 1024 threads 1024 segments took the same time).
constexpr uint32_t kPrologueWaves = 4;
constexpr uint32_t kRunTiles = 16;
static_assert(kRows >= 64 && kRows <= 128, "a wave holds the row counts of a tile, two per lane");

// Inclusive prefix sum over the wave's 64 lanes on the VALU's data-parallel
// primitives (no LDS round trips): row shifts by 1, 2, 4 and 8 scan each row
// of 16 lanes (a lane with no source adds 0), then the broadcasts of lane 15
// into rows 1 and 3 and of lane 31 into rows 2 and 3 carry the row totals up.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}

// The sum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(x), 63);
}

// Exclusive prefix sum of v over the workgroup in thread order; *total gets
// the sum of all.  wsum: one LDS word per wave.
__device__ uint32_t block_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t x = wave_incl_scan(v);
  __syncthreads();  // wsum is free
  if (lane == 63u) wsum[wave] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (uint32_t w = 0; w < blockDim.x / 64u; w++) {
    const uint32_t c = wsum[w];
    before += w < wave ? c : 0u;
    all += c;
  }
  *total = all;
  return before + x - v;
}

// Exclusive prefix sums of three values at once (one pass of barriers).
__device__ uint3 block_scan3(uint3 v, uint3* wsum, uint3* total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint3 x = make_uint3(wave_incl_scan(v.x), wave_incl_scan(v.y), wave_incl_scan(v.z));
  __syncthreads();  // wsum is free
  if (lane == 63u) wsum[wave] = x;
  __syncthreads();
  uint3 before = make_uint3(0u, 0u, 0u), all = make_uint3(0u, 0u, 0u);
  for (uint32_t w = 0; w < blockDim.x / 64u; w++) {
    const uint3 c = wsum[w];
    if (w < wave) {
      before.x += c.x;
      before.y += c.y;
      before.z += c.z;
    }
    all.x += c.x;
    all.y += c.y;
    all.z += c.z;
  }
  *total = all;
  return make_uint3(before.x + x.x - v.x, before.y + x.y - v.y, before.z + x.z - v.z);
}

// The expansion of a table with at most one segment per thread whose tiles are
// all cut alike (fewer tiles than CUs) or not at all: three barriers instead of
// eight, and no walk over runs.  Returns false, with nothing written, when the
// tail cut applies.  What it writes is what expand_tables says.  The waves work
// out the sums, the cut and the queue's class starts each for itself.  Bound by
// the latency of its phases.  Prologue, before and after: one 16 MiB segment
// (256 pieces, one thread placed them) 22.6 -> 6.3 us, 1024 segments of one tile
// 14.4 -> 12.1 us.
__device__ bool expand_short(const SegBrief* brief, uint32_t n, const ExpandArgs& x) {
  struct Rec {  // a segment's whole tiles: all of those before it, then its own
    uint32_t f0, p0, c0, nc, tb, nt, user, rank_rem;
  };
  __shared__ uint32_t cursor[kRows + 1];
  __shared__ uint4 sum1[kExpandThreads / 64];
  __shared__ uint3 sum2[kExpandThreads / 64];
  __shared__ Rec rec[kExpandThreads];
  const uint32_t tid = threadIdx.x, threads = blockDim.x, lane = tid & 63u, wave = tid >> 6, waves = threads >> 6;
  const bool have = tid < n;
  uint2 b = make_uint2(0u, 0u);
  if (have) b = ((const uint2*)brief)[tid];
  for (uint32_t i = tid; i <= (uint32_t)kRows; i += threads) cursor[i] = 0u;
  const uint32_t m = b.x, user = b.y;
  const bool small = have && m <= x.small_max, tiled = have && !small;
  const uint32_t nt = tiled ? tiles_in(m) : 0u, r = tiled ? tile_rows_of(m, nt - 1u) : 0u;
  const uint32_t scan_t = wave_incl_scan(nt);
  const unsigned long long smalls = __ballot(small);
  const uint32_t rows = wave_sum(tiled ? (nt - 1u) * kRows + r : 0u);
  const bool lng = __any(nt > 1u || r > (uint32_t)kPieceRows);
  if (lane == 63u) sum1[wave] = make_uint4(scan_t, (uint32_t)__popcll(smalls), rows, lng ? 1u : 0u);
  __syncthreads();

  uint32_t tb = scan_t - nt, sm = (uint32_t)__popcll(smalls & ((1ull << lane) - 1ull));
  uint32_t n_tiles = 0, rows_all = 0, any_long = 0;
  for (uint32_t v = 0; v < waves; v++) {
    const uint4 c = sum1[v];
    if (v < wave) tb += c.x, sm += c.y;
    n_tiles += c.x;
    rows_all += c.z;  // (read only with fewer tiles than CUs, when it is small)
    any_long |= c.w;
  }
  const bool fine = n_tiles < x.cus;
  if (!fine && any_long) return false;
  uint32_t p = fine ? (rows_all + x.cus - 1u) / x.cus : (uint32_t)kRows;
  if (p == 0u || p > (uint32_t)kRows) p = kRows;  // nothing is cut
  const uint32_t per = (uint32_t)kRows / p, rem = (uint32_t)kRows % p;
  const uint32_t whole = r == (uint32_t)kRows ? nt : nt - (nt ? 1u : 0u);
  const uint32_t nc = p < (uint32_t)kRows ? whole : 0u, nf = whole - nc;
  const bool part = r > 0u && r < (uint32_t)kRows, part_cut = part && r > p;
  const uint32_t part_pieces = part_cut ? r / p : 0u, part_len = part_cut ? r % p : part ? r : 0u;
  if (have) {
    x.tile_base[tid] = tb;
    if (x.seg_cut) x.seg_cut[tid] = nt == 1u && (nc || part_cut) ? 1u : 0u;
    if (small) x.small_list[sm] = tid;
  }
  if (tid == 0u) x.tile_base[n] = n_tiles;
  uint32_t rank_part = 0, rank_rem = 0;
  if (part_len) rank_part = atomicAdd(&cursor[part_len], 1u);
  if (nc && rem) rank_rem = atomicAdd(&cursor[rem], nc);
  const uint32_t np = nc * per + part_pieces;
  const uint3 sc = make_uint3(wave_incl_scan(nf), wave_incl_scan(np), wave_incl_scan(nc));
  if (lane == 63u) sum2[wave] = sc;
  __syncthreads();

  uint3 at = make_uint3(sc.x - nf, sc.y - np, sc.z - nc), all = make_uint3(0u, 0u, 0u);
  for (uint32_t v = 0; v < waves; v++) {
    const uint3 c = sum2[v];
    if (v < wave) at.x += c.x, at.y += c.y, at.z += c.z;
    all.x += c.x, all.y += c.y, all.z += c.z;
  }
  // class starts, longest first: lane k holds rows kRows - k and kRows - 64 - k
  const uint32_t ka = kRows - lane, kb = kRows - 64u - lane;
  const bool has_b = kRows > 64 + (int)lane;
  const uint32_t na = cursor[ka] + (ka == (uint32_t)kRows ? all.x : 0u) + (ka == p ? all.y : 0u);
  const uint32_t nb = has_b ? cursor[kb] + (kb == p ? all.y : 0u) : 0u;
  const uint32_t ia = wave_incl_scan(na), ib = (uint32_t)__builtin_amdgcn_readlane((int)ia, 63) + wave_incl_scan(nb);
  const uint32_t ents = (uint32_t)__builtin_amdgcn_readlane((int)ib, 63);
  auto start = [&](uint32_t len) -> uint32_t {
    const int k = (int)((uint32_t)kRows - len);
    const uint32_t a = __shfl(ia - na, k & 63), c = __shfl(ib - nb, k & 63);
    return k < 64 ? a : c;
  };
  const uint32_t piece_at = start(p), rem_at = rem ? start(rem) : 0u, part_at = start(part_len ? part_len : 1u);
  auto put = [&](uint32_t pos, uint32_t g0, uint32_t seg, uint32_t t, uint32_t r0, uint32_t r1, uint32_t u) {
    if (pos < x.cap) x.order[pos] = TileEnt{g0 + t, seg, t | (r0 << 16) | (r1 << 24), u};
  };
  if (part_len) {
    // an uncut partial tile, or the lowest piece of a cut one
    const uint32_t r1 = part_cut ? (uint32_t)kRows - part_pieces * p : (uint32_t)kRows;
    put(part_at + (part_len == p ? all.y : 0u) + rank_part, tb, tid, nt - 1u, part_cut && r1 > p ? r1 - p : 0u, r1, user);
  }
  if (all.x | all.y) {
    // whole tiles and pieces, spread over the threads: each finds its segment
    // by binary search over what the segments before it have
    rec[tid] = Rec{at.x, at.y, at.z, nc, tb, nt, user, rank_rem};
    __syncthreads();
    auto find = [&](uint32_t j, auto&& first) -> uint32_t {
      uint32_t lo = 0, hi = n;
      while (hi - lo > 1u) {
        const uint32_t mid = (lo + hi) >> 1;
        if (first(rec[mid]) <= j)
          lo = mid;
        else
          hi = mid;
      }
      return lo;
    };
    for (uint32_t j = tid; j < all.x; j += threads) {
      const uint32_t i = find(j, [](const Rec& q) { return q.f0; });
      const Rec q = rec[i];
      put(j, q.tb, i, q.nc + (j - q.f0), 0u, kRows, q.user);
    }
    for (uint32_t j = tid; j < all.y; j += threads) {
      const uint32_t i = find(j, [](const Rec& q) { return q.p0; });
      const Rec q = rec[i];
      const uint32_t d = j - q.p0, t = d / per;
      const uint32_t k = t < q.nc ? d % per : d - q.nc * per;
      put(piece_at + j, q.tb, i, t < q.nc ? t : q.nt - 1u, kRows - (k + 1u) * p, kRows - k * p, q.user);
    }
    if (rem)
      for (uint32_t j = tid; j < all.z; j += threads) {
        const uint32_t i = find(j, [](const Rec& q) { return q.c0; });
        const Rec q = rec[i];
        put(rem_at + (rem == p ? all.y : 0u) + q.rank_rem + (j - q.c0), q.tb, i, j - q.c0, 0u, rem, q.user);
      }
  }
  for (uint32_t k = ents + tid; k < x.cap; k += threads) x.order[k] = TileEnt{kNoTile, 0u, 0u, 0u};
  if (tid == 0u && x.n_ents) *x.n_ents = ents;
  return true;
}

// Expansion by the calling workgroup (all its threads call it), from the
// per-segment brief records (the source may be host memory).  A one-tile
// segment whose tile is cut gets seg_cut = 1 (every segment gets its 0 or 1,
// where seg_cut is given).
// The per-segment values the walks need sit in LDS for up to kInfoLds
// segments, else in x.info.
constexpr uint32_t kInfoLds = 1024;

__device__ void expand_tables(const SegBrief* brief, uint32_t n, const ExpandArgs& x) {
  if (n <= blockDim.x && expand_short(brief, n, x)) return;
  __shared__ uint32_t hist[kRows + 1];    // tiles by rows
  __shared__ uint32_t cursor[kRows + 1];  // entries by rows run, then the next free slot of each
  __shared__ uint32_t wsum[kExpandThreads / 64];
  __shared__ uint3 wsum3[kExpandThreads / 64];
  __shared__ uint32_t first_seg[kExpandThreads];  // segment of each thread's first run
  __shared__ SegInfo info_lds[kInfoLds];
  __shared__ unsigned long long rows_all;
  __shared__ uint32_t c_piece, c_from, c_take, c_left, c_fine, c_ents, c_full_at, c_piece_at;
  const uint32_t tid = threadIdx.x, nt_ = blockDim.x, lane = tid & 63u;
  SegInfo* info = n <= kInfoLds ? info_lds : x.info;
  for (uint32_t i = tid; i <= (uint32_t)kRows; i += nt_) hist[i] = cursor[i] = 0u;
  first_seg[tid] = 0xFFFFFFFFu;
  if (tid == 0) rows_all = 0ull;

  // the brief records, two per 16-byte load, several loads in flight per
  // thread (the source may be host memory); flags as the descriptors have them
  {
    const uint4* src = (const uint4*)brief;
    const uint32_t n16 = (n + 1) / 2;
    constexpr int kInFlight = 8;
    auto note = [&](uint32_t i, uint32_t m, uint32_t user) {
      const bool small = m <= x.small_max;
      info[i].m = m;
      info[i].flags = small ? kSegSmall : (m <= kTileBlocks ? kSegOneTile : 0u);
      info[i].user = user;
      if (x.seg_cut) x.seg_cut[i] = 0u;
    };
    for (uint32_t i0 = tid; i0 < n16; i0 += kInFlight * nt_) {
      uint4 q[kInFlight];
#pragma unroll
      for (int k = 0; k < kInFlight; k++)
        if (i0 + k * nt_ < n16) q[k] = src[i0 + k * nt_];
#pragma unroll
      for (int k = 0; k < kInFlight; k++) {
        const uint32_t i = i0 + k * nt_;
        if (i >= n16) break;
        note(2 * i, q[k].x, q[k].y);
        if (2 * i + 1 < n) note(2 * i + 1, q[k].z, q[k].w);
      }
    }
  }
  __syncthreads();

  // segments [s0, s1) of this thread: count tiles, rows, small segments and runs
  const uint32_t per = (n + nt_ - 1) / nt_;
  const uint32_t s0 = min(n, tid * per), s1 = min(n, s0 + per);
  uint32_t my_tiles = 0, my_small = 0, my_runs = 0, my_whole = 0;
  unsigned long long my_rows = 0;
  for (uint32_t s = s0; s < s1; s++) {
    const uint32_t m = info[s].m;
    if (info[s].flags & kSegSmall) {
      my_small++;
      continue;
    }
    const uint32_t nt = tiles_in(m), r = tile_rows_of(m, nt - 1);
    my_tiles += nt;
    my_runs += (nt + kRunTiles - 1) / kRunTiles;
    my_rows += (unsigned long long)(nt - 1) * kRows + r;
    my_whole += nt - 1;
    atomicAdd(&hist[r], 1u);
  }
  // the whole tiles below each segment's first tile, and the rows, once per
  // wave.  The rows are read only with fewer tiles than CUs, when no thread
  // has 2^20 of them; capped there, the sums stay within 32 bits.
  my_whole = wave_sum(my_whole);
  const uint32_t rows_w = wave_sum((uint32_t)min(my_rows, 1ull << 20));
  if (lane == 0u) {
    if (my_whole) atomicAdd(&hist[kRows], my_whole);
    if (rows_w) atomicAdd(&rows_all, (unsigned long long)rows_w);
  }
  uint3 tot;
  const uint3 base0 = block_scan3(make_uint3(my_tiles, my_small, my_runs), wsum3, &tot);
  const uint32_t tb0 = base0.x, sm0 = base0.y, rn0 = base0.z;
  const uint32_t n_tiles = tot.x, n_runs = tot.z;
  const uint32_t per_r = (n_runs + nt_ - 1) / nt_;  // runs per thread
  {
    uint32_t tb = tb0, sm = sm0, rn = rn0;
    for (uint32_t s = s0; s < s1; s++) {
      x.tile_base[s] = tb;
      info[s].tb = tb;
      info[s].rb = rn;
      const SegInfo v = info[s];
      if (v.flags & kSegSmall) {
        x.small_list[sm++] = s;
        continue;
      }
      const uint32_t nt = tiles_in(v.m), nr = (nt + kRunTiles - 1) / kRunTiles;
      // this segment's runs fall in the run ranges of threads rn / per_r ..
      // (rn + nr - 1) / per_r; the lowest such segment starts a thread's range
      for (uint32_t c = rn / per_r; c <= (rn + nr - 1) / per_r; c++) atomicMin(&first_seg[c], s);
      tb += nt;
      rn += nr;
    }
  }
  if (tid == 0) x.tile_base[n] = n_tiles;
  __syncthreads();  // hist, rows_all, first_seg and the segment values complete

  // the cut (wave 0): with enough tiles, every tile of at least `from` rows
  // and the first `left` tiles of `take` rows, counted from the longest down
  // to at most cus tiles
  if (tid < 64u) {
    uint32_t piece = 0, from = kRows + 1, take = 0, left = 0, fine = 0;
    if (n_tiles > 0 && n_tiles < x.cus) {
      const unsigned long long p = (rows_all + x.cus - 1) / x.cus;
      if (p < (unsigned long long)kRows) {
        piece = (uint32_t)p;
        fine = 1;
      }
    } else if (n_tiles > 0) {
      piece = kPieceRows;
      // lane k holds rows kRows - k and kRows - 64 - k (those above kPieceRows)
      constexpr uint32_t kSpan = (uint32_t)(kRows - kPieceRows);
      static_assert(kSpan <= 128, "two row counts per lane");
      const uint32_t ra = kRows - lane, rb = kRows - 64u - lane;
      const uint32_t ha = lane < kSpan ? hist[ra] : 0u, hb = lane + 64u < kSpan ? hist[rb] : 0u;
      const uint32_t ia = wave_incl_scan(ha);  // tiles of at least ra rows
      const uint32_t tot_a = (uint32_t)__builtin_amdgcn_readlane((int)ia, 63);
      const uint32_t ib = tot_a + wave_incl_scan(hb);
      // from = the least row count whose tiles and all longer ones fit in cus
      const unsigned long long fa = __ballot(lane < kSpan && ia <= x.cus);
      const unsigned long long fb = __ballot(lane + 64u < kSpan && ib <= x.cus);
      uint32_t fit = 0;  // tiles of at least `from` rows
      if (fb) {
        const uint32_t k = 63u - (uint32_t)__clzll(fb);  // the highest lane: the fewest rows
        from = kRows - 64u - k;
        fit = (uint32_t)__builtin_amdgcn_readlane((int)ib, (int)k);
      } else if (fa) {
        const uint32_t k = 63u - (uint32_t)__clzll(fa);
        from = kRows - k;
        fit = (uint32_t)__builtin_amdgcn_readlane((int)ia, (int)k);
      }
      left = x.cus - fit;
      if (left) {
        // the longest row count below from that has tiles (above kPieceRows)
        const unsigned long long ta = __ballot(lane < kSpan && ra < from && ha > 0u);
        const unsigned long long tb = __ballot(lane + 64u < kSpan && rb < from && hb > 0u);
        if (ta)
          take = kRows + 1u - (uint32_t)__ffsll((unsigned long long)ta);
        else if (tb)
          take = kRows - 63u - (uint32_t)__ffsll((unsigned long long)tb);
      }
    }
    if (tid == 0) {
      c_piece = piece;
      c_from = from;
      c_take = take;
      c_left = take ? left : 0u;
      c_fine = fine;
    }
  }
  __syncthreads();
  const uint32_t piece = c_piece, from = c_from, take = c_take, left = c_left;
  const bool fine = c_fine != 0;

  // rank in tile order of each segment's first tile of `take` rows
  auto takes_of = [&](uint32_t m, uint32_t nt) -> uint32_t {
    return (take == (uint32_t)kRows ? nt - 1 : 0u) + (tile_rows_of(m, nt - 1) == take ? 1u : 0u);
  };
  if (left) {
    uint32_t mine = 0, all;
    for (uint32_t s = s0; s < s1; s++)
      if (!(info[s].flags & kSegSmall)) mine += takes_of(info[s].m, tiles_in(info[s].m));
    uint32_t rank = block_scan(mine, wsum, &all);
    for (uint32_t s = s0; s < s1; s++) {
      info[s].tk = rank;
      if (!(info[s].flags & kSegSmall)) rank += takes_of(info[s].m, tiles_in(info[s].m));
    }
    __syncthreads();
  }
  // The tiles of a segment are t = 0 .. nt - 1 from its end; all have kRows
  // rows but the first, t = nt - 1, which has r1 rows.  A run [t0, t1) holds
  // nf whole tiles (t < fe), of which the first nc are cut, and maybe the
  // partial first tile.
  struct RunPlan {
    uint32_t nf, nc;  // whole tiles, cut whole tiles (a prefix of them)
    bool part;        // holds the partial first tile
    bool part_cut;
    uint32_t r1;      // its rows
  };
  auto plan_run = [&](const SegInfo& v, uint32_t t0, uint32_t t1) -> RunPlan {
    RunPlan q;
    const uint32_t nt = tiles_in(v.m);
    q.r1 = tile_rows_of(v.m, nt - 1);
    const uint32_t fe = q.r1 == (uint32_t)kRows ? nt : nt - 1;  // whole tiles are t < fe
    const uint32_t fend = min(t1, fe);
    q.nf = fend > t0 ? fend - t0 : 0u;
    // whole tiles are cut: all of them (a fine cut, or kRows >= from), else
    // those whose rank among the tiles of `take` = kRows rows is below left
    if (fine || (uint32_t)kRows >= from) {
      q.nc = q.nf;
    } else if (take == (uint32_t)kRows && left > v.tk) {
      const uint32_t cend = min(fend, left - v.tk);  // t < left - tk
      q.nc = cend > t0 ? cend - t0 : 0u;
    } else {
      q.nc = 0;
    }
    q.part = q.r1 < (uint32_t)kRows && nt - 1 >= t0 && nt - 1 < t1;
    q.part_cut = q.part && (fine ? q.r1 > piece : (q.r1 >= from || (q.r1 == take && left > v.tk)));
    return q;
  };

  // runs [r_lo, r_hi) of this thread, from the segment holding run r_lo;
  // visit(s, v, t0, t1): tiles t0 .. t1 - 1 of segment s (values v)
  const uint32_t r_lo = min(n_runs, tid * per_r), r_hi = min(n_runs, r_lo + per_r);
  auto walk = [&](auto&& visit) {
    if (r_lo >= r_hi) return;
    uint32_t s = first_seg[tid];
    SegInfo v = info[s];
    uint32_t run = r_lo - v.rb;  // run of s
    for (uint32_t k = r_lo; k < r_hi; k++) {
      while ((v.flags & kSegSmall) || run * kRunTiles >= tiles_in(v.m)) {  // on to the next tiled segment
        s++;
        run = 0;
        v = info[s];
      }
      const uint32_t t0 = run * kRunTiles;
      visit(s, v, t0, min(tiles_in(v.m), t0 + kRunTiles));
      run++;
    }
  };
  // Count the entries by the rows each runs.  Uncut whole tiles (kRows
  // rows) and whole pieces get slots by thread order, which is tile order;
  // the other lengths (partial tiles, the remainders of cut tiles) by LDS
  // atomics.
  const uint32_t rem_full = piece ? (uint32_t)kRows % piece : 0u;  // remainder piece of a cut whole tile
  uint32_t my_full = 0, my_pieces = 0;
  walk([&](uint32_t s, const SegInfo& v, uint32_t t0, uint32_t t1) {
    const RunPlan q = plan_run(v, t0, t1);
    my_full += q.nf - q.nc;
    if (q.nc) {
      my_pieces += q.nc * ((uint32_t)kRows / piece);
      if (rem_full) atomicAdd(&cursor[rem_full], q.nc);
    }
    if (q.part) {
      if (!q.part_cut) {
        atomicAdd(&cursor[q.r1], 1u);
      } else {
        my_pieces += q.r1 / piece;
        if (q.r1 % piece) atomicAdd(&cursor[q.r1 % piece], 1u);
      }
    }
    // a one-tile segment has one run: this thread owns its entry
    if (x.seg_cut && (v.flags & kSegOneTile) && (q.nc || q.part_cut)) x.seg_cut[s] = 1u;
  });
  uint3 tot2;
  const uint3 b2 = block_scan3(make_uint3(my_full, my_pieces, 0u), wsum3, &tot2);
  const uint32_t full0 = b2.x, piece0 = b2.y, n_full = tot2.x, n_pieces = tot2.y;
  if (tid < 64u) {  // start of each length's run, longest first: lane k holds rows kRows - k and kRows - 64 - k
    const uint32_t ka = kRows - lane, kb = kRows - 64u - lane;
    const bool has_b = kRows > 64 + (int)lane;
    const uint32_t ca = cursor[ka] + (ka == (uint32_t)kRows ? n_full : 0u) + (ka == piece ? n_pieces : 0u);
    const uint32_t cb = has_b ? cursor[kb] + (kb == piece ? n_pieces : 0u) : 0u;
    const uint32_t ia = wave_incl_scan(ca), tot_a = (uint32_t)__builtin_amdgcn_readlane((int)ia, 63);
    const uint32_t ib = tot_a + wave_incl_scan(cb);
    // the atomics of a length start after its slots taken in thread order
    cursor[ka] = ia - ca + (ka == (uint32_t)kRows ? n_full : 0u) + (ka == piece ? n_pieces : 0u);
    if (has_b) cursor[kb] = ib - cb + (kb == piece ? n_pieces : 0u);
    if (ka == (uint32_t)kRows) c_full_at = ia - ca;  // first slot of the whole tiles
    if (ka == piece) c_piece_at = ia - ca;           // first slot of the whole pieces
    if (has_b && kb == piece) c_piece_at = ib - cb;
    if (lane == 63u) c_ents = ib;
  }
  __syncthreads();
  uint32_t at_full = c_full_at + full0, at_piece = (n_pieces ? c_piece_at : 0u) + piece0;
  walk([&](uint32_t s, const SegInfo& v, uint32_t t0, uint32_t t1) {
    const RunPlan q = plan_run(v, t0, t1);
    const uint32_t user = v.user, g0 = v.tb;
    auto put = [&](uint32_t pos, uint32_t t, uint32_t r0, uint32_t r1) {
      if (pos < x.cap) x.order[pos] = TileEnt{g0 + t, s, t | (r0 << 16) | (r1 << 24), user};
    };
    // pieces [r1 - piece, r1) from the tile's end down; the lowest may start
    // below the tile's first row lo
    auto pieces = [&](uint32_t t, uint32_t rows) {
      const uint32_t lo = (uint32_t)kRows - rows;
      for (uint32_t r1 = kRows; r1 > lo; r1 -= min(r1, piece)) {
        const uint32_t r0 = r1 > piece ? r1 - piece : 0u, len = r1 - max(r0, lo);
        put(len == piece ? at_piece++ : atomicAdd(&cursor[len], 1u), t, r0, r1);
      }
    };
    // a cut whole tile: kRows / piece whole pieces, then the remainder, if any
    const uint32_t per_tile = q.nc ? (uint32_t)kRows / piece : 0u;
    for (uint32_t t = t0; t < t0 + q.nc; t++) {
      for (uint32_t k = 0; k < per_tile; k++) put(at_piece++, t, kRows - (k + 1) * piece, kRows - k * piece);
      if (rem_full) put(atomicAdd(&cursor[rem_full], 1u), t, 0u, rem_full);
    }
    for (uint32_t t = t0 + q.nc; t < t0 + q.nf; t++) put(at_full++, t, 0u, kRows);
    if (q.part) {
      const uint32_t t = tiles_in(v.m) - 1;
      if (q.part_cut)
        pieces(t, q.r1);
      else
        put(atomicAdd(&cursor[q.r1], 1u), t, 0u, kRows);
    }
  });
  const uint32_t ents = c_ents;
  for (uint32_t k = ents + tid; k < x.cap; k += nt_) x.order[k] = TileEnt{kNoTile, 0u, 0u, 0u};
  if (tid == 0 && x.n_ents) *x.n_ents = ents;
}

// The expansion alone, for the library's test hook.
__global__ __launch_bounds__(kExpandThreads) void k_expand(const SegBrief* brief, uint32_t n, ExpandArgs x) {
  expand_tables(brief, n, x);
}

// ---------------------------------------------------------------------------
// First kernel of a call.  It copies the call's staged tables (descriptors,
// zero ranges, zeroed queue head, block ids) from the mapped host ring into
// device scratch, zeroes the tile partials, settles every segment's first
// verdict -- with labels, the owner check (OWNER_MIXED iff some row label
// differs from the segment's user; the sentinels never equal a user), else
// OK.  With an expansion,
// workgroup 0 builds the tile tables and the work queue meanwhile from the
// brief records; the other workgroups read descriptors and block ids where
// the copy reads them, so no part waits on another.
// ---------------------------------------------------------------------------
struct PrologueArgs {
  uint4* dst;
  const uint4* src;  // nullptr: the tables are in dst already
  size_t n16;        // 16-byte words of staged tables
  const SegDesc* segs;  // where the descriptors are readable now (src or dst)
  uint32_t n;
  const uint32_t* labels;
  const uint32_t* bids;
  int32_t* verdicts;
  uint4* zero;
  uint32_t n_zero;
  ChunkTable chunks;
  bool by_wave;
  bool expand;
  const SegBrief* brief;  // where the brief records are readable now
  ExpandArgs x;
};

__global__ __launch_bounds__(kPrologueThreads) void k_prologue(PrologueArgs a) {
  const bool ex = a.expand && a.n > 0;
  if (ex && blockIdx.x == 0) {
    expand_tables(a.brief, a.n, a.x);
    if (gridDim.x > 1) return;  // the other workgroups do the rest
    __syncthreads();
  }
  // the other workgroups (all of them without an expansion, or workgroup 0
  // after it when it is alone, which launch_prologue does not ask for: as an
  // early return for good the same call of 1024 segments takes 68.4 us, so 67.8)
  const bool sep = ex && gridDim.x > 1;
  const uint32_t wg = sep ? blockIdx.x - 1 : blockIdx.x, n_wg = sep ? gridDim.x - 1 : gridDim.x;
  const size_t gsz = (size_t)n_wg * blockDim.x, me = (size_t)wg * blockDim.x + threadIdx.x;
  // A segment per wave (by_wave: few rows per segment) or per workgroup.  The
  // descriptors may be in host memory, about 2 us away: a wave reads one in one
  // access, the first one before anything else, and writes its copy.
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const bool mine = a.verdicts && (!a.by_wave || wave < kPrologueWaves);
  const uint32_t first = a.by_wave ? wg * kPrologueWaves + wave : wg, step = a.by_wave ? n_wg * kPrologueWaves : n_wg;
  auto descriptor = [&](uint32_t s) { return lane < 16u ? ((const uint32_t*)(a.segs + s))[lane] : 0u; };
  uint32_t dv = mine && first < a.n ? descriptor(first) : 0u;
  if (a.src)
    for (size_t i = (a.verdicts ? (size_t)a.n * (sizeof(SegDesc) / 16) : 0) + me; i < a.n16; i += gsz)
      a.dst[i] = a.src[i];
  for (size_t i = me; i < a.n_zero; i += gsz) a.zero[i] = make_uint4(0u, 0u, 0u, 0u);
  // paged calls: where each chunk is.  The segments' chunks follow each other
  // as their blocks do in the block-id array: chunk c is chunk c % per_block of
  // block c / per_block.
  const ChunkTable& ct = a.chunks;
  for (uint64_t c = me; c < ct.n; c += gsz) {
    const uint64_t j = ct.n >> 32 ? c / ct.per_block : (uint32_t)c / (uint32_t)ct.per_block;
    const uint64_t i = c - j * ct.per_block;  // layer and part
    const uint64_t l = ct.n >> 32 ? i / ct.parts : (uint32_t)i / ct.parts;
    ct.off[c] = l * ct.layer_stride + (uint64_t)a.bids[j] * ct.block_stride + (i - l * ct.parts) * ct.part_stride;
  }
  if (!mine) return;
  for (uint32_t s = first; s < a.n; s += step) {
    if (s != first) dv = descriptor(s);
    if (a.src && lane < 16u && (a.by_wave || wave == 0u)) ((uint32_t*)((SegDesc*)a.dst + s))[lane] = dv;
    auto word = [&](size_t at) { return lane_word(dv, (int)(at / 4)); };
    auto word2 = [&](size_t at) { return (uint64_t)word(at + 4) << 32 | word(at); };
    const uint32_t user = word(offsetof(SegDesc, user));
    int bad = 0;
    if (a.labels) {
      const uint64_t rb = word2(offsetof(SegDesc, row_begin)), rc = word2(offsetof(SegDesc, row_count));
      const uint32_t r0 = a.by_wave ? lane : threadIdx.x, rs = a.by_wave ? 64u : blockDim.x;
      // Eight labels in flight per thread; past the end the last one again.
      // One at a time, a segment's labels took a memory latency each: 256
      // prompts of 16-8192 tokens, whose workgroups read up to 32 labels per
      // thread, 38.1 us per call, now 34.8.
      for (uint64_t r = r0; r < rc; r += 8ull * rs) {
        uint64_t at[8];
        uint32_t l[8];
#pragma unroll
        for (uint32_t k = 0; k < 8u; k++) at[k] = rb + min(r + k * (uint64_t)rs, rc - 1u);
        if (a.bids) {
          uint32_t id[8];
#pragma unroll
          for (int k = 0; k < 8; k++) id[k] = a.bids[at[k]];
#pragma unroll
          for (int k = 0; k < 8; k++) at[k] = id[k];
        }
#pragma unroll
        for (int k = 0; k < 8; k++) l[k] = a.labels[at[k]];
#pragma unroll
        for (int k = 0; k < 8; k++) bad |= l[k] != user;
      }
      bad = a.by_wave ? __any(bad) : __syncthreads_or(bad);
    }
    if ((a.by_wave ? lane : threadIdx.x) == 0u) a.verdicts[s] = bad ? kVerdictOwnerMixed : kVerdictOk;
  }
}

// ---------------------------------------------------------------------------
// Zero-fill of uncovered rows and of rejected segments.
// ---------------------------------------------------------------------------
// Zero-fill of uncovered rows and (open) of segments whose verdict is not OK.
// The host cuts ranges into pieces of at most kZeroPieceBytes; a workgroup
// takes whole pieces, so nothing loops over all ranges per thread.
__global__ __launch_bounds__(256) void k_zero_ranges(uint8_t* out, const ZeroRange* __restrict__ rs, uint32_t n,
                                                     const int32_t* __restrict__ verdicts) {
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const ZeroRange z = rs[i];
    if (z.seg >= 0 && verdicts[z.seg] == kVerdictOk) continue;
    uint8_t* p = out + z.off;
    uint64_t head = (16u - ((uintptr_t)p & 15u)) & 15u;
    if (head > z.len) head = z.len;
    for (uint64_t b = threadIdx.x; b < head; b += blockDim.x) p[b] = 0;
    const uint64_t mid = (z.len - head) / 16u;
    uint4* q = (uint4*)(p + head);
    for (uint64_t k = threadIdx.x; k < mid; k += blockDim.x) q[k] = make_uint4(0u, 0u, 0u, 0u);
    for (uint64_t b = head + 16u * mid + threadIdx.x; b < z.len; b += blockDim.x) p[b] = 0;
  }
}

__global__ __launch_bounds__(256) void k_wipe(uint8_t* p, size_t bytes) {
  const size_t gsz = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < bytes; i += gsz) p[i] = 0;
}


// ---------------------------------------------------------------------------
// Per-token encryption (token || nonce as one block under the owner's key,
// the end-of-sequence token as the all-0xFF block).  The work is cut into runs
// of tokens of one segment, whose records the host writes (16 B: all that the
// kernel needs of a segment); they may be in host memory.  A workgroup of 64
// threads takes 64 tokens, and 2^shift workgroups share a run.  Outputs of
// uncovered tokens were zeroed before this launch.
//
// Bound by latency: the record, then keys and tokens, then 14 AES rounds.  With
// a prologue kernel that copied the descriptors to the device and a search for
// each workgroup's segment there, a call on 1024 segments of 1-4 tokens took
// 24.3 us, now 17.1, which is the host's share; 64 prompts of 128-2048 tokens
// 16.1, now 14.5.
// With the table's loads waited for one by one and ahead of the record's, and the
// token's ahead of the nonce's, the kernel itself took 12.9 us for 2,588 tokens
// of 1,024 users, now 8.3.
// ---------------------------------------------------------------------------
template <bool DECRYPT>
__global__ __launch_bounds__(kTokenChunk) void k_tokens(const TokenRun* __restrict__ runs, uint32_t n_runs,
                                                        uint32_t shift,
                                                        const uint64_t* __restrict__ tokens,
                                                        const uint64_t* __restrict__ nonces,
                                                        const uint8_t* __restrict__ blocks_in,
                                                        uint8_t* __restrict__ blocks_out,
                                                        uint64_t* __restrict__ tokens_out,
                                                        uint64_t* __restrict__ nonces_out, uint64_t eos_token,
                                                        KeyTableDev kt) {
  __shared__ uint32_t tab[256];
  __shared__ uint32_t isb[64];
  static_assert(kTokenChunk == 64, "one wave per workgroup: a round-key word per lane");
  const uint32_t lane = threadIdx.x;
  // the table and the first record (there are at least as many as workgroups)
  // are under way together
  uint32_t tv[4], iv = 0;
#pragma unroll
  for (uint32_t k = 0; k < 4u; k++) tv[k] = (DECRYPT ? c_aes.td0 : c_aes.te0)[64u * k + lane];
  if (DECRYPT) iv = ((const uint32_t*)c_aes.inv_sbox)[lane];
  auto record = [&](uint64_t b) { return ((const uint32_t*)(runs + (b >> shift)))[lane & 3u]; };
  uint32_t rv = record(blockIdx.x);
#pragma unroll
  for (uint32_t k = 0; k < 4u; k++) tab[64u * k + lane] = tv[k];
  if (DECRYPT) isb[lane] = iv;
  rv = opaque(rv);  // loaded here: not moved behind the barrier
  __syncthreads();
  for (uint64_t b = blockIdx.x; b < (uint64_t)n_runs << shift; b += gridDim.x) {
    if (b != blockIdx.x) rv = record(b);
    const uint64_t row = (uint64_t)lane_word(rv, 1) << 32 | lane_word(rv, 0);
    const uint32_t user = lane_word(rv, 2), count = lane_word(rv, 3);
    const uint32_t i0 = kTokenChunk * ((uint32_t)b & ((1u << shift) - 1u)), i = i0 + lane;
    if (i0 >= count) continue;  // the run is shorter
    const uint32_t keys = (DECRYPT ? kt.dk : kt.rk)[64ull * user + lane];
    // The rounds take their keys from all lanes, so all lanes run them, past
    // the run's end on its last token again; only the stores are masked.
    const uint64_t r = row + min(i, count - 1u);
    if (!DECRYPT) {
      const uint64_t t = tokens[r], n = nonces[r];
      const uint32_t blk[4] = {(uint32_t)t, (uint32_t)(t >> 32), (uint32_t)n, (uint32_t)(n >> 32)};
      uint32_t o[4];
      aes256_encrypt_tab(keys, blk, o, tab);
      const uint32_t e = t == eos_token ? 0xFFFFFFFFu : 0u;
      if (i < count) *(uint4*)(blocks_out + 16ull * r) = make_uint4(o[0] | e, o[1] | e, o[2] | e, o[3] | e);
    } else {
      const uint4 c = *(const uint4*)(blocks_in + 16ull * r);
      const uint32_t blk[4] = {c.x, c.y, c.z, c.w};
      uint32_t p[4];
      aes256_decrypt_tab(keys, blk, p, tab, (const uint8_t*)isb);
      const bool eos = (c.x & c.y & c.z & c.w) == 0xFFFFFFFFu;
      if (i < count) {
        tokens_out[r] = eos ? eos_token : (uint64_t)p[0] | ((uint64_t)p[1] << 32);
        if (nonces_out) nonces_out[r] = eos ? 0ull : (uint64_t)p[2] | ((uint64_t)p[3] << 32);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Open: zero the output of segments that failed, tile by tile.  A workgroup
// takes whole tiles of kTileBlocks blocks (the GCM kernel's tiles, found
// through tile_base), so the work per workgroup is bounded.  Contiguous
// output (chunk_off == nullptr): every segment whose verdict is not OK.
// Through block tables: only requests that failed authentication -- their
// blocks passed the label check, so they are the request's own; a request
// rejected by the label check writes nothing.  Nothing to do unless a tag
// failed (*any_failed): in contiguous output the tile kernel has zeroed the
// segments that the label check rejected.
__global__ __launch_bounds__(256) void k_zero_failed(const uint32_t* __restrict__ any_failed,
                                                     const SegDesc* __restrict__ segs, uint32_t n,
                                                     const uint32_t* __restrict__ tile_base, uint32_t n_tiles,
                                                     const int32_t* __restrict__ verdicts,
                                                     const uint64_t* __restrict__ chunk_off, uint8_t* base,
                                                     uint32_t chunk_shift) {
  if (*any_failed == 0u) return;
  const uint64_t cmask = (1ull << chunk_shift) - 1;
  for (uint32_t g = blockIdx.x; g < n_tiles; g += gridDim.x) {
    uint32_t lo = 0, hi = n;  // tile_base[lo] <= g < tile_base[hi]
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (tile_base[mid] <= g)
        lo = mid;
      else
        hi = mid;
    }
    const int32_t v = verdicts[lo];
    if (chunk_off ? v != kVerdictAuthFail : v == kVerdictOk) continue;
    const uint64_t m = segs[lo].nblocks;
    const uint64_t t = g - tile_base[lo];
    // tiles are aligned to the end of the segment, as in k_gcm_tiles
    const uint64_t end = m - t * (uint64_t)kTileBlocks;
    const uint64_t begin = end > kTileBlocks ? end - kTileBlocks : 0;
    if (chunk_off) {
      const uint64_t c0 = segs[lo].chunk0;
      for (uint64_t i = begin + threadIdx.x; i < end; i += blockDim.x)
        *(uint4*)(base + chunk_off[c0 + (i >> chunk_shift)] + ((i & cmask) << 4)) = make_uint4(0u, 0u, 0u, 0u);
    } else {
      const uint64_t len = segs[lo].len;
      uint8_t* p = base + segs[lo].byte_off;
      for (uint64_t i = begin + threadIdx.x; i < end; i += blockDim.x) {
        const uint64_t rem = len - 16ull * i;
        store_block(p + 16ull * i, u128_zero(), rem >= 16 ? 16u : (uint32_t)rem);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Key-table setup.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_key_sched(const uint8_t* __restrict__ keys, KeyTableDev kt) {
  const uint32_t u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= kt.n_users) return;
  uint32_t rk[60];
  aes256_key_schedule(keys + 32ull * u, rk, c_aes);
  for (int i = 0; i < 60; i++) kt.rk[64ull * u + i] = rk[i];
  for (int i = 60; i < 64; i++) kt.rk[64ull * u + i] = 0u;
  uint32_t dk[60];
  aes256_dec_key_schedule(rk, dk);
  for (int i = 0; i < 60; i++) kt.dk[64ull * u + i] = dk[i];
  for (int i = 60; i < 64; i++) kt.dk[64ull * u + i] = 0u;
  const uint32_t zero[4] = {0u, 0u, 0u, 0u};
  uint32_t h[4];
  aes256_encrypt_words(rk, zero, h, c_aes);
  for (int i = 0; i < 4; i++) kt.h[4ull * u + i] = h[i];
}

constexpr uint32_t kPowersPerUser = kHPowers + kFinLanes + 1 + kHxLanes + kRows;

__global__ __launch_bounds__(256) void k_key_powers(KeyTableDev kt) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t u = idx / kPowersPerUser;
  const uint32_t j = (uint32_t)(idx % kPowersPerUser);
  if (u >= kt.n_users) return;
  const u128 h = ld_u128((const uint4*)(kt.h + 4ull * u));
  if (j < (uint32_t)kHPowers) {
    st_u128(kt.pow_h + u * kHPowers + j, gf_pow(h, j));
  } else if (j < (uint32_t)(kHPowers + kFinLanes)) {
    const uint32_t l = j - kHPowers;
    st_u128(kt.pow_ht + u * kFinLanes + l, gf_pow(h, (uint64_t)l * kTileBlocks));
  } else if (j == (uint32_t)(kHPowers + kFinLanes)) {
    st_u128(kt.pow_hlt + u, gf_pow(h, (uint64_t)kFinLanes * kTileBlocks));
  } else if (j < (uint32_t)(kHPowers + kFinLanes + 1 + kHxLanes)) {
    const uint32_t k = j - (kHPowers + kFinLanes + 1);
    st_u128(kt.pow_hxl + u * kHxLanes + k, gf_mul(h, gf_xpow_elem(64 + (int)k)));
  } else {
    const uint32_t k = j - (kHPowers + kFinLanes + 1 + kHxLanes);
    st_u128(kt.pow_hr + u * kRows + k, gf_pow(h, (uint64_t)k * kThreads));
  }
}

// Nibble tables of M = H^1024 and H^512 (k_gcm_tiles with one team, with
// two): entry [q][v] = (v placed at GCM bits 4q..4q+3, MSB first) * M, built
// from the four products x^(4q+k) * M.
__global__ __launch_bounds__(256) void k_key_gtab(KeyTableDev kt) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t u = idx / 64u;
  const int q = (int)(idx % 32u);
  const uint32_t two = (uint32_t)(idx / 32u) & 1u;
  if (u >= kt.n_users) return;
  const u128 mm = gf_pow(ld_u128((const uint4*)(kt.h + 4ull * u)), two ? (uint64_t)kThreads / 2 : (uint64_t)kThreads);
  uint4* tab = kt.gtab + (u * 2u + two) * 512u;
  u128 b[4];
  for (int k = 0; k < 4; k++) b[k] = gf_mul(gf_xpow_elem(4 * q + k), mm);
  for (int v = 0; v < 16; v++) {
    u128 e = u128_zero();
    for (int k = 0; k < 4; k++)
      if (v & (8 >> k)) e = u128_xor(e, b[k]);
    st_u128(tab + (uint64_t)q * 16u + v, e);
  }
}

// ---------------------------------------------------------------------------
// Launch wrappers.
// ---------------------------------------------------------------------------
static inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

hipError_t launch_key_setup(const uint8_t* keys_dev, KeyTableDev kt, hipStream_t s) {
  hipLaunchKernelGGL(k_key_sched, dim3(cdiv(kt.n_users, 64)), dim3(64), 0, s, keys_dev, kt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_key_powers, dim3(cdiv((uint64_t)kt.n_users * kPowersPerUser, 256)), dim3(256), 0, s, kt);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_key_gtab, dim3(cdiv((uint64_t)kt.n_users * 64u, 256)), dim3(256), 0, s, kt);
  return hipGetLastError();
}



template <int TEAMS>
static hipError_t launch_tiles(const GcmArgs& a, int mode, uint32_t g, hipStream_t s) {
  switch (mode) {
    case 0: hipLaunchKernelGGL((k_gcm_tiles<0, TEAMS>), dim3(g), dim3(kThreads), 0, s, a); break;
    case kModeOpen: hipLaunchKernelGGL((k_gcm_tiles<kModeOpen, TEAMS>), dim3(g), dim3(kThreads), 0, s, a); break;
    case kModeGather: hipLaunchKernelGGL((k_gcm_tiles<kModeGather, TEAMS>), dim3(g), dim3(kThreads), 0, s, a); break;
    case kModeOpen | kModeScatter:
      hipLaunchKernelGGL((k_gcm_tiles<kModeOpen | kModeScatter, TEAMS>), dim3(g), dim3(kThreads), 0, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gcm_tiles(const GcmArgs& a, int mode, uint32_t grid, uint32_t teams, hipStream_t s) {
  if (a.n_ents == 0) return hipSuccess;
  const uint32_t g = a.n_ents < grid ? a.n_ents : grid;
  return teams == 2 ? launch_tiles<2>(a, mode, g, s) : launch_tiles<1>(a, mode, g, s);
}

hipError_t launch_gcm_small(const GcmArgs& a, bool open, hipStream_t s) {
  if (a.n_small == 0) return hipSuccess;
  if (open)
    hipLaunchKernelGGL(k_small<true>, dim3(a.n_small), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL(k_small<false>, dim3(a.n_small), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_zero_ranges(uint8_t* out, const ZeroRange* r, uint32_t n, const int32_t* verdicts, uint32_t grid,
                              hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (grid > n) grid = n;
  hipLaunchKernelGGL(k_zero_ranges, dim3(grid), dim3(256), 0, s, out, r, n, verdicts);
  return hipGetLastError();
}

hipError_t launch_tokens(const TokenRun* runs, uint32_t n_runs, uint32_t shift, bool decrypt, const uint64_t* tokens,
                         const uint64_t* nonces, const uint8_t* blocks_in, uint8_t* blocks_out, uint64_t* tokens_out,
                         uint64_t* nonces_out, uint64_t eos_token, KeyTableDev kt, hipStream_t s) {
  if (n_runs == 0) return hipSuccess;
  const uint64_t n_wg = (uint64_t)n_runs << shift;
  const uint32_t grid = n_wg < 65535u ? (uint32_t)n_wg : 65535u;
  if (decrypt)
    hipLaunchKernelGGL(k_tokens<true>, dim3(grid), dim3(kTokenChunk), 0, s, runs, n_runs, shift, tokens, nonces, blocks_in,
                       blocks_out, tokens_out, nonces_out, eos_token, kt);
  else
    hipLaunchKernelGGL(k_tokens<false>, dim3(grid), dim3(kTokenChunk), 0, s, runs, n_runs, shift, tokens, nonces, blocks_in,
                       blocks_out, tokens_out, nonces_out, eos_token, kt);
  return hipGetLastError();
}

hipError_t launch_zero_failed(const uint32_t* any_failed, const SegDesc* segs, uint32_t n_segs, const uint32_t* tile_base, uint32_t n_tiles,
                              const int32_t* verdicts, const uint64_t* chunk_off, uint8_t* base, uint32_t chunk_shift,
                              uint32_t grid, hipStream_t s) {
  if (n_segs == 0 || n_tiles == 0) return hipSuccess;
  if (grid > n_tiles) grid = n_tiles;
  hipLaunchKernelGGL(k_zero_failed, dim3(grid), dim3(256), 0, s, any_failed, segs, n_segs, tile_base, n_tiles,
                     verdicts, chunk_off, base, chunk_shift);
  return hipGetLastError();
}


hipError_t launch_expand(const SegBrief* brief, uint32_t n_segs, const ExpandArgs& x, hipStream_t s) {
  if (n_segs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_expand, dim3(1), dim3(kExpandThreads), 0, s, brief, n_segs, x);
  return hipGetLastError();
}

hipError_t launch_prologue(void* dst, const void* src, size_t bytes, uint32_t n_segs, uint64_t rows, uint64_t bids_off,
                           const uint32_t* labels, int32_t* verdicts, uint4* zero, uint32_t n_zero, uint64_t brief_off, const ExpandArgs* ex,
                           const ChunkTable* chunks, hipStream_t s) {
  if (bytes & 15u) return hipErrorInvalidValue;
  const size_t n16 = src ? bytes / 16 : 0;
  const bool expand = ex != nullptr && n_segs > 0;
  if (n16 == 0 && !verdicts && n_zero == 0 && !expand) return hipSuccess;
  if (n16 && (((uintptr_t)dst | (uintptr_t)src) & 15u)) return hipErrorInvalidValue;
  if (expand && (brief_off & 15u || brief_off + 8ull * (n_segs + 1) > bytes)) return hipErrorInvalidValue;
  const uint8_t* rd = src ? (const uint8_t*)src : (const uint8_t*)dst;  // where the tables are readable now
  const uint32_t threads = n_segs <= 256u ? 256u : (uint32_t)kPrologueThreads;
  uint64_t grid = cdiv(n16 > n_zero ? n16 : n_zero, threads);
  // Segments of up to 64 rows on average take a wave each, so that 1024 of
  // them need 256 workgroups; longer ones a workgroup, whose threads read the
  // labels of a KV segment (thousands of rows) in a few steps.  A long segment
  // among many short ones is one wave's, too, 512 labels at a time: 1024 segments
  // of one row and one of 60,000 are checked in 34.7 us per call, 16,384 and one
  // of a million in 806 (with a workgroup for every segment, one label per thread
  // at a time, 36.5 and 1093).
  const bool by_wave = rows <= 64ull * n_segs;
  if (chunks && cdiv(chunks->n, threads) > grid) grid = cdiv(chunks->n, threads);
  const uint64_t per_wg = by_wave ? kPrologueWaves : 1;
  if (verdicts && cdiv(n_segs, per_wg) > grid) grid = cdiv(n_segs, per_wg);
  if (grid > 512u) grid = 512u;
  if (grid == 0) grid = 1;
  if (expand) grid += 1;  // workgroup 0 expands the segment table
  PrologueArgs a{};
  a.dst = (uint4*)dst;
  a.src = (const uint4*)src;
  a.n16 = n16;
  a.segs = (const SegDesc*)rd;
  a.n = n_segs;
  a.labels = labels;
  a.bids = bids_off == kNoBids ? nullptr : (const uint32_t*)(rd + bids_off);
  a.verdicts = verdicts;
  a.zero = zero;
  a.n_zero = n_zero;
  if (chunks) a.chunks = *chunks;
  a.by_wave = by_wave;
  a.expand = expand;
  if (expand) {
    a.x = *ex;
    a.brief = (const SegBrief*)(rd + brief_off);
  }
  hipLaunchKernelGGL(k_prologue, dim3((uint32_t)grid), dim3(threads), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fixed workspace of gift_seal_noalloc.  Each device holds its own copy of
// the array at its own address; host code never uses the array's name (a
// host-side stand-in), only the address hipGetSymbolAddress gives for the
// current device, looked up once per device at set-up.
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

static std::mutex g_scratch_mu;
static uint8_t* g_scratch_addr[kStaticScratchDevices] = {nullptr};

hipError_t static_scratch_setup(int dev) {
  if (dev < 0 || dev >= kStaticScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (g_scratch_addr[dev]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (ptr == nullptr || ((uintptr_t)ptr & 255u)) return hipErrorInvalidSymbol;
  g_scratch_addr[dev] = (uint8_t*)ptr;
  return hipSuccess;
}

uint8_t* static_scratch(int dev) {
  if (dev < 0 || dev >= kStaticScratchDevices) return nullptr;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  return g_scratch_addr[dev];
}

hipError_t launch_wipe(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  uint32_t grid = cdiv(bytes, 256u * 16u);
  if (grid > 4096u) grid = 4096u;
  hipLaunchKernelGGL(k_wipe, dim3(grid), dim3(256), 0, s, (uint8_t*)p, bytes);
  return hipGetLastError();
}

}  // namespace gift
