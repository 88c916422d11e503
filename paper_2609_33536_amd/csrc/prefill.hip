// Chunked-prefill attention over a mixed-fidelity paged prefix for gfx950
// (paper §3.2: BASE blocks are read as their high bytes with a zero low
// byte; App. A: a prefill chunk attends its cached prefix and, causally,
// itself).
//
// A workgroup of 4 waves serves one (sequence, KV head, tile of query
// tokens); a wave works on 32 query "columns" -- (token, head-in-group) pairs.
// The work unit is one pair of blocks, 32 keys (the missing second block of
// a lone last one is masked).  On 32x32x16 matrix cores, per unit:
//   S^T (32 keys x 32 columns) = K (32 x 128) . Q^T, 8 products;
//     lane l holds column l % 32 and keys 8(r/4) + 4(l/32) + r%4, r < 16.
//   online softmax over those 16 scores (+ the partner lane l ^ 32);
//   O^T (128 dims x 32 columns) += V^T . P^T, for P's 16-bit head and its
//     16-bit remainder (P keeps ~16 significant bits), 4 dim tiles x 2
//     key steps x 2.  The P operand of key step k is the lane's own scores
//     r = 8k .. 8k+7, so key index 8(l/32) + i of step k stands for key
//     16k + 8(i/4) + 4(l/32) + i%4; the V^T operand follows the same order.
// V^T operands come straight from LDS with the transposing read
// ds_read_b64_tr_b16: within each 16-lane group it hands lane j element j of
// the rows the group's lanes point at (row 4a + j/4, element j%4), so pointing
// lane 4a + b at key a, dims d + 4b .. gives lane j keys a = 0..3 of dim d + j.
// Column c sees keys p < lim(c) = prefix + (its chunk index) + 1.
//
// Every unit lies in LDS as 16-bit words whatever its kind, so one branch-free
// body serves TARGET and BASE blocks and 8-bit pools: TARGET words are loaded
// straight to their place; bytes (BASE, or 8-bit TARGET) and nibbles (8-bit
// BASE) are loaded raw and widened in place, once per workgroup (a wave widens
// the quarter that it loaded).  When every wave fetched and widened the BASE
// operands for itself, a unit cost a wave 182 vector, 110 scalar and 21 branch
// instructions (its 24 products aside); now 147, 59 and 9.
//
// Two kernels:
//   prefill_kernel        4 waves x 32 columns share every unit (pipelined, or
//                         in rounds of 4 units over contexts of at most 8);
//   prefill_split_kernel  4 waves share 32 columns and take every fourth unit
//                         each: small launches, which leave most CUs idle.
#include <cstdlib>
#include <type_traits>

#include "attn_device.h"
#include "prefill_plan.h"

namespace ekv {
namespace {

constexpr int kPfWaves = 4;
constexpr int kPfCols = 32;       // query columns per wave
constexpr int kPfWindow = 64;     // pairs per metadata window: one per lane

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short i16x4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4v* lds_i16x4;

template <typename T> struct Mma32;
template <> struct Mma32<Bf16> {
  static __device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   c, 0, 0, 0);
  }
};
template <> struct Mma32<Fp16> {
  static __device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b),
                                                  c, 0, 0, 0);
  }
};

// Two probabilities -> packed 16-bit heads and packed 16-bit remainders
// (head + remainder = p to ~16 significant bits).  bf16: the head is the
// upper half of the fp32 word (truncation), one byte permute for the pair.
template <typename T>
__device__ __forceinline__ void split_p(float p0, float p1, uint32_t& hi, uint32_t& lo);

template <>
__device__ __forceinline__ void split_p<Bf16>(float p0, float p1, uint32_t& hi, uint32_t& lo) {
  const uint32_t x0 = __float_as_uint(p0), x1 = __float_as_uint(p1);
  hi = perm(x1, x0, 0x07060302u);   // upper halves: x0 -> low word, x1 -> high word
  // both remainders rounded to nearest-even in one packed conversion
  const f32x2v rem = {p0 - __uint_as_float(x0 & 0xffff0000u), p1 - __uint_as_float(x1 & 0xffff0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(rem, bf16x2v));
}
template <>
__device__ __forceinline__ void split_p<Fp16>(float p0, float p1, uint32_t& hi, uint32_t& lo) {
  // one packed conversion for the heads (to nearest); p - head is exact, so one
  // mixed-precision fused multiply-add rounds each remainder into its half
  typedef _Float16 f16x2v __attribute__((ext_vector_type(2)));
  const f16x2v h = __builtin_convertvector((f32x2v{p0, p1}), f16x2v);
  const f16x2v r = {(_Float16)__builtin_fmaf(-1.0f, (float)h[0], p0), (_Float16)__builtin_fmaf(-1.0f, (float)h[1], p1)};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, r);
}

// 8 nibbles (element e in byte e/2, low nibble for even e) -> 8 bytes,
// each nibble in the high half of its byte (an executed 4-bit BASE value).
__device__ __forceinline__ u32x2 widen_nibbles(uint32_t w) {
  const uint32_t even = (w << 4) & 0xF0F0F0F0u, odd = w & 0xF0F0F0F0u;
  return u32x2{perm(odd, even, 0x05010400u), perm(odd, even, 0x07030602u)};
}

// max of three floats.  Written for the compiler, not as inline assembly:
// its operands come straight from the matrix cores, and only the compiler
// inserts the wait states a vector instruction needs before it may read an
// MFMA result (inline assembly would read the registers while the products
// are still being written).
__device__ __forceinline__ float max3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

// v *= f, written for the compiler: the accumulators come straight from the
// matrix cores, and only the compiler inserts the wait states a vector
// instruction needs before it reads an MFMA result.  (On gfx950 the
// multiplies stay in the accumulators' own registers: no copies on the
// common path that skips the rescale.)
__device__ __forceinline__ void scale_in_place(f32x16& v, float f) {
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] *= f;
}

// Workgroup barrier that also orders this wave's LDS accesses.  On gfx950
// s_barrier does not wait for the wave's outstanding LDS operations, and
// the compiler adds no wait before a bare s_barrier: an LDS write issued
// before it (the widened 8-bit tiles) could land after another wave has
// passed the barrier and read the old bytes, and an LDS read still in
// flight could see a slot that the ring's next load has begun to refill.
// s_waitcnt lgkmcnt(0) completes every LDS access of the wave first.  The
// ring's direct-to-LDS loads are vector memory operations, waited for with
// explicit counts before the barrier that publishes a slot.
__device__ __forceinline__ void barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A unit's slot in LDS: the K rows of both blocks, then the V rows, in groups
// of 4 rows: 1 KiB (one direct-to-LDS load: 64 lanes x 16 bytes) and 16 bytes
// of padding.  In a group, 16-byte chunk c of row r sits at position
// 16 (c / 4) + 4 r + c % 4.  So a K read (16 rows, one chunk) and a transposing
// V read (4 rows x 4 chunks of one group) touch 16 distinct 16-byte positions
// of a 256-byte bank cycle, and the head-dim step, the dim tile and the key
// step of every read are constant offsets from one address per lane.
constexpr int kGroup = 1024 + 16;
constexpr int kTilePf = 4 * kGroup;       // 16 rows
constexpr int kSlotPf = 4 * kTilePf;      // K of both blocks, V of both
constexpr int kPlanePf = 2 * kTilePf;     // V's offset in a slot

// Offset of row group 2 half of block `member`: quarter q = 2 member + half of
// a plane, 8 rows, is loaded and widened as one piece.
__device__ __forceinline__ constexpr uint32_t quarter_offset(int q) { return (q >> 1) * kTilePf + 2 * (q & 1) * kGroup; }

// One direct-to-LDS load: lane l's 16 bytes at base + off go to lds + 16 l.
// Inline assembly (it writes no register) keeps it out of the compiler's wait
// insertion, which would wait for every load in flight before each transposing
// LDS read; the kernels wait with explicit counts.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is named as clobbered although the compiler never allocates it)
__device__ __forceinline__ void dma16(uint64_t base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Loads and widening of quarters.  A unit costs a quarter kLoads loads (2 of
// K, 2 of V; half for 8-bit pools) whatever its kind, so that constant counts
// wait for it: a 16-bit BASE quarter has half the bytes and loads them twice
// (the copy is overwritten when the quarter is widened), an 8-bit BASE quarter
// of 512 bytes twice with the two halves of the wave.
template <bool F8>
struct Stager {
  static constexpr int kLoads = F8 ? 2 : 4;
  static constexpr int kTileP = F8 ? kTileBytes / 2 : kTileBytes;   // a (plane, head) tile in the pool
  uint32_t src_t, src_b, src_n;   // source offsets in a quarter: words, bytes, nibbles
  uint32_t raw_n, dst;            // nibbles' place in the raw quarter; this lane's words in the widened one
  int row;                        // row of the quarter whose 16-element chunk this lane widens
  uint64_t v_off;                 // K plane -> V plane in the pool

  __device__ __forceinline__ Stager(int lane, int num_kv_heads) {
    src_t = ((lane >> 2) & 3) * 256 + 64 * (lane >> 4) + 16 * (lane & 3);
    // lane -> (row, chunk) so that 16 consecutive lanes write 16 distinct
    // positions of a bank cycle when they widen
    row = (lane >> 1) & 7;
    const int chunk = 2 * (lane >> 4) + (lane & 1);
    src_b = row * kHeadDim + 16 * chunk;
    src_n = 16 * (lane & 31);
    raw_n = row * (kHeadDim / 2) + 8 * chunk;
    dst = (row >> 2) * kGroup + 256 * (chunk >> 1) + 64 * (row & 3) + 32 * (chunk & 1);
    v_off = (uint64_t)num_kv_heads * kTileP;
  }
  // Quarter q of a unit, tile: the K tile of the quarter's block (a BASE
  // pair's: the packed tile), slot: the unit's slot (LDS address).
  __device__ __forceinline__ void load(uint64_t tile, bool base, int q, uint32_t slot) const {
    const uint32_t to = slot + quarter_offset(q);
    const uint64_t packed = tile + (uint32_t)(q >> 1) * (kTileP / 2);
    if constexpr (F8) {
      const uint32_t off = base ? src_n : src_b;
      const uint64_t src = base ? packed + (q & 1) * 8 * (kHeadDim / 2) : tile + (q & 1) * 8 * kHeadDim;
      dma16(src, off, to);
      dma16(src + v_off, off, to + kPlanePf);
    } else {
      const uint32_t off = base ? src_b : src_t;
      const uint64_t src = base ? packed + (q & 1) * 8 * kHeadDim : tile + (q & 1) * 8 * 2 * kHeadDim;
      const uint64_t src2 = src + (base ? 0 : 1024);
      dma16(src, off, to);
      dma16(src2, off, to + kGroup);
      dma16(src + v_off, off, to + kPlanePf);
      dma16(src2 + v_off, off, to + kPlanePf + kGroup);
    }
  }
  // After quarter q has landed: bytes or nibbles -> words in place (every
  // lane's reads precede the wave's writes), and zero V rows for keys at or
  // past `valid` (their slots may hold anything, and 0 * NaN would poison
  // the products).  key0: the unit's first key.
  __device__ __forceinline__ void widen(char* slot, bool base, int q, int key0, int valid, int lane) const {
    char* at = slot + quarter_offset(q);
    if (F8 || base) {
      u32x4 raw[2];
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        if (F8 && base) {
          const u32x2 x = *reinterpret_cast<const u32x2*>(at + pl * kPlanePf + raw_n);
          const u32x2 lo = widen_nibbles(x.x), hi = widen_nibbles(x.y);
          raw[pl] = u32x4{lo.x, lo.y, hi.x, hi.y};
        } else {
          raw[pl] = *reinterpret_cast<const u32x4*>(at + pl * kPlanePf + 16 * lane);
        }
      }
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        *reinterpret_cast<u32x4*>(at + pl * kPlanePf + dst) = expand_base8(raw[pl].xy);
        *reinterpret_cast<u32x4*>(at + pl * kPlanePf + dst + 16) = expand_base8(raw[pl].zw);
      }
    }
    if (key0 + 2 * kPage > valid && key0 + 8 * q + row >= valid) {
      *reinterpret_cast<u32x4*>(at + kPlanePf + dst) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(at + kPlanePf + dst + 16) = u32x4{0u, 0u, 0u, 0u};
    }
  }
};

// The block table of one sequence in windows of 64 pairs: lane l holds the K
// tile addresses of both blocks of pair w0 + l, and a mask the pairs' modes, so
// that a unit's loads read their addresses from a lane, with no LDS or memory
// round trip.  The next window's entries are fetched a window ahead.
template <bool ELASTIC, bool F8>
struct PairTable {
  const int32_t* row;
  const uint8_t* tags;
  int base_lo = 0, base_hi = 0;   // BASE pairs by boundaries (when the tags are not used)
  bool use_tags = false;
  int nblk, units, num_blocks;
  uint64_t pool, block_bytes;
  int w0 = 0;
  uint64_t addr0 = 0, addr1 = 0, base_mask = 0;   // the current window
  int next0 = 0, next1 = 0;                       // the next one, as read
  bool next_base = false;

  __device__ __forceinline__ PairTable(const PrefillArgs& a, int s, int kvh, int nblk_, int lane) : nblk(nblk_) {
    row = a.bt + (size_t)s * a.max_blocks;
    tags = a.tags ? a.tags + (size_t)s * a.max_blocks : nullptr;
    units = (nblk + 1) >> 1;
    num_blocks = a.num_blocks;
    block_bytes = (uint64_t)2 * a.num_kv_heads * Stager<F8>::kTileP;
    pool = reinterpret_cast<uint64_t>(a.pool) + (uint64_t)kvh * Stager<F8>::kTileP;
    if constexpr (ELASTIC) {
      int b0 = -1, b1 = -1;
      if (a.bounds) {
        b0 = a.bounds[2 * s];
        b1 = a.bounds[2 * s + 1];
      }
      if (b0 >= 0) {
        base_lo = b0;
        base_hi = b1;
      } else if (tags) {
        use_tags = true;
      }
    }
    fetch(0, lane);
    enter();
    if (units > kPfWindow) fetch(kPfWindow, lane);
  }
  __device__ __forceinline__ void fetch(int from, int lane) {
    const int p = from + lane;
    next0 = next1 = 0;
    next_base = false;
    if (p < units) {
      next0 = row[2 * p];
      next1 = 2 * p + 1 < nblk ? row[2 * p + 1] : next0;   // a lone last block stands in for the missing one (masked)
      if constexpr (ELASTIC) next_base = use_tags ? tags[2 * p] != 0 : (p >= base_lo && p < base_hi);
    }
  }
  __device__ __forceinline__ void enter() {
    const int b0 = (unsigned)next0 < (unsigned)num_blocks ? next0 : 0;   // never leave the pool
    const int b1 = (unsigned)next1 < (unsigned)num_blocks ? next1 : 0;
    addr0 = pool + (uint64_t)(uint32_t)b0 * block_bytes;
    addr1 = next_base ? addr0 : pool + (uint64_t)(uint32_t)b1 * block_bytes;   // (a BASE pair lies in its first block)
    base_mask = __builtin_amdgcn_ballot_w64(next_base);
  }
  // unit u (nondecreasing over calls); its mode
  __device__ __forceinline__ bool seek(int u, int lane) {
    if (u >= w0 + kPfWindow) {
      w0 = u & ~(kPfWindow - 1);
      enter();
      if (w0 + kPfWindow < units) fetch(w0 + kPfWindow, lane);
    }
    return ELASTIC && ((base_mask >> (u & (kPfWindow - 1))) & 1) != 0;
  }
  __device__ __forceinline__ uint64_t tile(int u, int member) const {
    const uint64_t a = member ? addr1 : addr0;
    const int l = u & (kPfWindow - 1);
    uint64_t at = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(a >> 32), l) << 32) |
                  (uint32_t)__builtin_amdgcn_readlane((uint32_t)a, l);
    // A scalar register that a vector instruction writes needs 5 wait states
    // before a vector memory instruction reads it; the hardware does not check,
    // and the compiler does not look into dma16.  These 3, and the 2 before
    // dma16's load, for all the loads that use the address (waiting in every
    // load cost the 8B chunked prefill 1 %).
    asm("s_nop 2" : "+s"(at));
    return at;
  }
};

// One wave's 32 query columns of a (sequence, KV head).
template <typename T, int G>
struct Columns {
  u32x4 q[8];              // Q^T operands: dims 16 k + 8 h .. + 7
  size_t row;              // this lane's query row (element offset in q and out)
  int lim, lim_all;        // keys this lane's column sees; keys every column sees
  bool ok;
  float c_scale;           // |scale| log2(e): a negative scale negates the queries instead (exact)
  f32x16 o[4];
  float m = -__builtin_inff(), l = 0.f;   // reference max (log2 units, the same in lanes l and l ^ 32), this lane's sum

  // first column col0 of the sequence's chunk; q0, nq: its rows; prefix, len: its keys
  __device__ __forceinline__ Columns(const PrefillArgs& a, int kvh, int q0, int nq, int len, int col0, int lane) {
    const int col = col0 + (lane & 31), h = lane >> 5;
    const int tq = col / G, head = col % G, prefix = len - nq;
    ok = tq < nq;
    lim = ok ? min(len, prefix + tq + 1) : len;
    lim_all = min(len, prefix + col0 / G + 1);
    c_scale = fabsf(a.scale_log2);
    const uint32_t sign = a.scale_log2 < 0.f ? 0x80008000u : 0u;
    row = ((size_t)(q0 + (ok ? tq : 0)) * a.num_q_heads + (size_t)kvh * G + head) * kHeadDim;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      q[k] = ok ? (*reinterpret_cast<const u32x4*>(a.q + row + 16 * k + 8 * h) ^ sign) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int t = 0; t < 4; ++t) o[t] = f32x16{};
  }
  __device__ __forceinline__ f32x16 scores(const u32x4 (&k)[8]) const {
    f32x16 s = f32x16{};
#pragma unroll
    for (int i = 0; i < 8; ++i) s = Mma32<T>::mma(k[i], q[i], s);
    return s;
  }
  // Scores enter the softmax as s * c in log2 units (c is returned).  Units
  // that every column sees whole fold c into the max and the exponent; the
  // others scale first and then set masked keys to -inf, so that a zero
  // scale never multiplies an infinity (0 * -inf is NaN).
  __device__ __forceinline__ float mask(f32x16& s, int key0, int h) const {
    if (key0 + 2 * kPage <= lim_all) return c_scale;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      s[r] = key0 + 8 * (r >> 2) + 4 * h + (r & 3) >= lim ? -__builtin_inff() : s[r] * c_scale;
    return 1.0f;
  }
  // Moves the reference max if some column's unit max exceeds it by more than
  // 2^8 (wave-uniform result); then *shift = old - new reference (log2).
  __device__ __forceinline__ bool advance(const f32x16& s, float c, float* shift) {
    const float m0 = max3(s[0], s[1], s[2]), m1 = max3(s[3], s[4], s[5]);
    const float m2 = max3(s[6], s[7], s[8]), m3 = max3(s[9], s[10], s[11]);
    const float m4 = max3(s[12], s[13], s[14]);
    float mx = max3(max3(m0, m1, m2), max3(m3, m4, s[15]), m0);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = __builtin_fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c;
    const bool moved = __builtin_amdgcn_ballot_w64(mx > m + 8.0f) != 0;
    const float to = moved ? __builtin_fmaxf(m, mx) : m;
    *shift = m - to;
    m = to;
    return moved;
  }
  // P = exp2(s c - ref) as 16-bit heads and remainders; returns the lane's sum.
  __device__ __forceinline__ float probabilities(const f32x16& s, float c, float ref, u32x4 (&hi)[2], u32x4 (&lo)[2]) const {
    float sum[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = fast_exp2(__builtin_fmaf(s[8 * ks + i], c, -ref));
      sum[ks] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      uint32_t wh[4], wl[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) split_p<T>(p[2 * i], p[2 * i + 1], wh[i], wl[i]);
      hi[ks] = u32x4{wh[0], wh[1], wh[2], wh[3]};
      lo[ks] = u32x4{wl[0], wl[1], wl[2], wl[3]};
    }
    return sum[0] + sum[1];
  }
  __device__ __forceinline__ void accumulate(const u32x4 (&v)[4], u32x4 p) {
#pragma unroll
    for (int t = 0; t < 4; ++t) o[t] = Mma32<T>::mma(v[t], p, o[t]);
  }
  __device__ __forceinline__ void rescale(float f) {
    l *= f;
#pragma unroll
    for (int t = 0; t < 4; ++t) scale_in_place(o[t], f);
  }
  __device__ __forceinline__ float total() const {   // the column's sum
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
};

// Dim tile t of a column's output: this lane holds dims 32 t + 8 u + 4 h .. + 3.
template <typename T>
__device__ __forceinline__ void store_tile(const PrefillArgs& a, size_t row, const f32x16& o, float inv, int t, int h) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const size_t idx = row + 32 * t + 8 * u + 4 * h;
    store_pair<T>(a.out, idx, o[4 * u] * inv, o[4 * u + 1] * inv, a.out_fp32);
    store_pair<T>(a.out, idx + 2, o[4 * u + 2] * inv, o[4 * u + 3] * inv, a.out_fp32);
  }
}

// Per-lane offsets of the K and V^T reads in a slot.
__device__ __forceinline__ uint32_t k_read_offset(int lane) {
  const int n = lane & 31;   // key row; chunk 2 k + h of step k
  return (n >> 4) * kTilePf + ((n >> 2) & 3) * kGroup + 64 * (n & 3) + 16 * (lane >> 5);
}
__device__ __forceinline__ uint32_t v_read_offset(int lane) {
  const int i = lane & 15, key = i >> 2, d = i & 3;
  return kPlanePf + (lane >> 5) * kGroup + 64 * key + 16 * (2 * ((lane >> 4) & 1) + (d >> 1)) + 8 * (d & 1);
}
__device__ __forceinline__ void read_k(const char* at, u32x4 (&k)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) k[i] = *reinterpret_cast<const u32x4*>(at + 256 * (i >> 1) + 32 * (i & 1));
}
__device__ __forceinline__ void read_v(const char* at, u32x4 (&v)[2][4]) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const char* p = at + ks * kTilePf + 256 * t;
      const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)p));
      const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)(p + 2 * kGroup)));
      v[ks][t] = u32x4{a.x, a.y, b.x, b.y};
    }
}

// A sequence's rows and keys, clamped into q, out and the table.
struct Extent {
  int q0, nq, len;
  __device__ __forceinline__ Extent(const PrefillArgs& a, int s) {
    q0 = min(max(a.cu_q[s], 0), a.total_q);
    nq = min(max(a.cu_q[s + 1], q0), a.total_q) - q0;
    len = max(0, min(a.seq_lens[s], a.max_blocks * kPage));
  }
  // keys that chunk row t sees, at least 1
  __device__ __forceinline__ int seen(int t) const { return max(1, min(len, len - nq + t + 1)); }
};

__device__ __forceinline__ PrefillPlace place(const PrefillArgs& a, int tiles) {
  return place_workgroup(blockIdx.x, blockIdx.y, gridDim.x, gridDim.y, tiles, a.num_kv_heads, a.batch, a.spread != 0);
}

// ---- 4 waves x 32 columns over shared units --------------------------------
// Software pipeline, one barrier a unit: the body of unit i runs the softmax of
// unit i while the matrix cores run the P.V products of unit i - 1 and the
// scores of unit i + 1 (both in the same basic block, so the compiler
// interleaves them), reads K of unit i + 1 and V of unit i, widens unit i + 2
// and issues the loads of unit i + 3.  4 slots, 66,560 B of LDS: two
// workgroups, two waves per SIMD (228-236 registers).
// Measured in one run against the kernel before (32-key units fetched and
// widened per wave, no pipeline), append of the chunk included: 8B chunked
// prefill (16 x (2048 prefix, half BASE, + 512), 32 / 8 heads, bf16) 537 ->
// 481 us; 8-bit pool, 2 x (8192 + 1024), 64 / 8 heads 958 -> 852 us; 3 short
// fp16 prompts 36 -> 28 us.
// What bounds it: matrix work under the power limit.  The kernel runs 1.5x the
// algorithmic flops (P's remainder); with random operands a plain 8192^3 bf16
// product reaches 1.2-1.3 PFLOP/s on this card (1.7 with zeros), which is
// ~370 us for this work, and leaving out the exponentials or the LDS reads
// changes the time by only 2-4 %.  Not kept: 64 columns per wave with one wave
// per SIMD (half the LDS reads, but a lone wave issues a vector instruction
// only every ~4.9 cycles: 4-6 % slower); the remainders p - head by
// v_dot2_f32_bf16 (fewer instructions, but they occupy the matrix pipe: 5 % slower).
constexpr int kPfRing = 4;
// Contexts of at most kPfFew units skip the pipeline, whose fill and drain (the
// loads past the last unit, a unit of products each before the first and after
// the last) cost more there than it hides: the ring is filled with up to 4 units
// at once, and a wave works through them without a barrier.  Measured (us, bf16,
// pipeline / rounds): 64 prompts of up to 16 rows, 16 / 16 heads 12.9 / 10.4, of up
// to 77 rows, 64 / 8 heads 47.8 / 44.7; 5-8 units, 16 x (200 + up to 77), 32 / 8
// heads 20.0 / 18.2, 8-bit, 64 / 8 heads 26.4 / 24.8.
constexpr int kPfFew = 8;

template <typename T, int G, bool ELASTIC, bool F8>
__global__ __launch_bounds__(64 * kPfWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_kernel(PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) char ring[kPfRing * kSlotPf];
  constexpr int kTileTok = kPfWaves * kPfCols / G;
  const int tiles = (a.max_q_len + kTileTok - 1) / kTileTok;
  const PrefillPlace at = place(a, tiles);
  const int s = at.seq, kvh = at.kv_head, tile = at.tile;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const Extent x(a, s);
  const int t_begin = tile * kTileTok;
  if (t_begin >= x.nq) return;   // uniform over the workgroup

  Columns<T, G> col(a, kvh, x.q0, x.nq, x.len, t_begin * G + wave * kPfCols, lane);
  const int nblk = (x.seen(min(x.nq, t_begin + kTileTok) - 1) + kPage - 1) / kPage;
  PairTable<ELASTIC, F8> table(a, s, kvh, nblk, lane);
  const int units = table.units;
  // the units this wave's own columns see (none if it has no column)
  const int t_wave = t_begin + wave * kPfCols / G;
  const int own_units = t_wave >= x.nq ? 0 : (x.seen(min(x.nq, t_wave + (kPfCols + G - 1) / G) - 1) + 31) >> 5;
  const int valid = min(x.len, nblk * kPage);   // V rows of keys at or past this are zeroed
  const Stager<F8> stager(lane, a.num_kv_heads);
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lds_ptr)&ring[0]);
  const char* k_at = ring + k_read_offset(lane);
  const char* v_at = ring + v_read_offset(lane);
  auto slot_of = [](int u) -> uint32_t { return (uint32_t)(u & (kPfRing - 1)) * kSlotPf; };

  int issued = 0;
  uint32_t modes = 0;       // bit 0: the unit issued last is BASE
  auto issue = [&]() {      // (past the last unit, its loads again, into a slot that nothing reads)
    const int u = min(issued, units - 1);
    const bool base = table.seek(u, lane);
    stager.load(table.tile(u, wave >> 1), base, wave, lds + slot_of(issued));
    modes = (modes << 1) | (base ? 1u : 0u);
    ++issued;
  };
  // this wave's quarter of unit u, when IN_FLIGHT units after it may still be loading
  auto stage = [&](int u, auto in_flight) {
    wait_loads<Stager<F8>::kLoads * decltype(in_flight)::value>();
    stager.widen(ring + slot_of(u), ELASTIC && ((modes >> (issued - 1 - u)) & 1u) != 0u, wave, 32 * u, valid, lane);
  };

  if (units <= kPfFew) {
#pragma unroll 1
    for (int u0 = 0; u0 < units; u0 += kPfRing) {
      const int u1 = min(units, u0 + kPfRing);
      if (u0 > 0) barrier();   // every wave is done with the ring
#pragma unroll 1
      for (int u = u0; u < u1; ++u) issue();
#pragma unroll 1
      for (int u = u0; u < u1; ++u) stage(u, std::integral_constant<int, 0>{});
      barrier();
#pragma unroll 1
      for (int u = u0; u < min(u1, own_units); ++u) {
        u32x4 k[8], v[2][4], hi[2], lo[2];
        read_k(k_at + slot_of(u), k);
        read_v(v_at + slot_of(u), v);
        f32x16 sc = col.scores(k);
        const float c = col.mask(sc, 32 * u, h);
        float shift;
        if (col.advance(sc, c, &shift)) col.rescale(fast_exp2(shift));
        col.l += col.probabilities(sc, c, col.m, hi, lo);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          col.accumulate(v[ks], hi[ks]);
          col.accumulate(v[ks], lo[ks]);
        }
      }
    }
  } else {
    u32x4 hi[2], lo[2], k[8], v[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      hi[ks] = lo[ks] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 4; ++t) v[ks][t] = u32x4{0u, 0u, 0u, 0u};
    }
    auto products = [&]() {   // O += V^T P^T of the unit whose P and V are in registers
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        col.accumulate(v[ks], hi[ks]);
        col.accumulate(v[ks], lo[ks]);
      }
    };
#pragma unroll 1
    for (int u = 0; u < kPfRing - 1; ++u) issue();
    stage(0, std::integral_constant<int, kPfRing - 2>{});
    stage(1, std::integral_constant<int, kPfRing - 3>{});
    barrier();
    read_k(k_at, k);
    f32x16 sc = col.scores(k);

#pragma unroll 1
    for (int i = 0; i < units; ++i) {
      barrier();   // units i and i + 1 are whole; unit i - 1's slot is free
      issue();
      if (i < own_units) {
        const float c = col.mask(sc, 32 * i, h);
        float shift;
        const bool moved = col.advance(sc, c, &shift);
        read_k(k_at + slot_of(i + 1), k);
        products();
        read_v(v_at + slot_of(i), v);
        const f32x16 next = col.scores(k);
        u32x4 nhi[2], nlo[2];
        float sum = col.probabilities(sc, c, col.m, nhi, nlo);
        // (kept in this block, beside the products: not sunk below the rescale's branch)
        asm volatile("" : "+v"(nhi[0]), "+v"(nhi[1]), "+v"(nlo[0]), "+v"(nlo[1]), "+v"(sum));
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          hi[ks] = nhi[ks];
          lo[ks] = nlo[ks];
        }
        sc = next;
        if (moved) col.rescale(fast_exp2(shift));   // (unit i - 1's products, under the old reference, are in)
        col.l += sum;
      }
      stage(i + 2, std::integral_constant<int, kPfRing - 3>{});
    }
    wait_loads<0>();   // no load may land after the workgroup has ended
    products();
  }

  const float inv = 1.0f / col.total();
  if (col.ok) {
#pragma unroll
    for (int t = 0; t < 4; ++t) store_tile<T>(a, col.row, col.o[t], inv, t, h);
  }
}

// ---- 4 waves share 32 columns and divide the units --------------------------
// A small chunk gives few workgroups of 128 columns, each a serial chain over
// its units (~0.7 us a unit, two LDS round trips, the matrix chain and the
// softmax among them) while most CUs idle.  Here a workgroup has 32 columns and
// wave w takes units w, w + 4, ...: a quarter of the chain, four times the
// workgroups.  A wave loads and widens its units alone (two slots of its own,
// no barrier in the loop); the waves' (o, m, l) are merged through LDS.
// Three fp16 prompts of 17-130 tokens over prefixes of up to 700: 28.8 -> 17.2 us;
// one 4715-token context + 3 rows, 32 / 8 heads: 92 -> 43.
template <typename T, int G, bool ELASTIC, bool F8>
__global__ __launch_bounds__(64 * kPfWaves) __attribute__((amdgpu_waves_per_eu(1, 1))) void prefill_split_kernel(PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) char ring[kPfWaves * 2 * kSlotPf];
  constexpr int kTileTok = kPfCols / G;
  const int tiles = (a.max_q_len + kTileTok - 1) / kTileTok;
  const PrefillPlace at = place(a, tiles);
  const int s = at.seq, kvh = at.kv_head, tile = at.tile;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const Extent x(a, s);
  const int t_begin = tile * kTileTok;
  if (t_begin >= x.nq) return;   // uniform over the workgroup

  Columns<T, G> col(a, kvh, x.q0, x.nq, x.len, t_begin * G, lane);
  const int nblk = (x.seen(min(x.nq, t_begin + kTileTok) - 1) + kPage - 1) / kPage;
  PairTable<ELASTIC, F8> table(a, s, kvh, nblk, lane);
  const int units = table.units;
  const int valid = min(x.len, nblk * kPage);   // V rows of keys at or past this are zeroed
  const Stager<F8> stager(lane, a.num_kv_heads);
  char* own = ring + wave * 2 * kSlotPf;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lds_ptr)own);
  const uint32_t k_at = k_read_offset(lane), v_at = v_read_offset(lane);
  constexpr int kUnitLoads = 4 * Stager<F8>::kLoads;

  bool base_of[2] = {false, false};   // the units in slots 0 and 1
  auto issue = [&](int u, int slot) {
    const bool base = table.seek(u, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) stager.load(table.tile(u, q >> 1), base, q, lds + slot * kSlotPf);
    base_of[slot] = base;
  };
  auto unit = [&](int u, int slot) {
    char* at = own + slot * kSlotPf;
    if (u + kPfWaves < units) wait_loads<kUnitLoads>();
    else wait_loads<0>();
#pragma unroll
    for (int q = 0; q < 4; ++q) stager.widen(at, base_of[slot], q, 32 * u, valid, lane);
    u32x4 k[8], v[2][4], hi[2], lo[2];
    read_k(at + k_at, k);
    read_v(at + v_at, v);
    f32x16 sc = col.scores(k);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read
    if (u + 2 * kPfWaves < units) issue(u + 2 * kPfWaves, slot);
    const float c = col.mask(sc, 32 * u, h);
    float shift;
    // (columns that see none of this wave's keys yet keep the reference -inf)
    if (col.advance(sc, c, &shift)) col.rescale(shift == shift ? fast_exp2(shift) : 1.0f);
    col.l += col.probabilities(sc, c, col.m == -__builtin_inff() ? 0.f : col.m, hi, lo);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      col.accumulate(v[ks], hi[ks]);
      col.accumulate(v[ks], lo[ks]);
    }
  };
  if (wave < units) issue(wave, 0);
  if (wave + kPfWaves < units) issue(wave + kPfWaves, 1);
#pragma unroll 1
  for (int u = wave; u < units; u += 2 * kPfWaves) {
    unit(u, 0);
    if (u + kPfWaves < units) unit(u + kPfWaves, 1);
  }

  // ---- merge: wave w sums dim tile w of the four waves ----
  const float l = col.total();
  barrier();   // every wave is done with the slots (its last loads have been waited for)
  f32x4* parts = reinterpret_cast<f32x4*>(ring);                                  // [wave][tile][4][lane]
  float2* ml = reinterpret_cast<float2*>(ring + kPfWaves * 16 * 64 * sizeof(f32x4));   // [wave][lane]
  ml[64 * wave + lane] = make_float2(col.m, l);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      parts[((wave * 4 + t) * 4 + r) * 64 + lane] =
          f32x4{col.o[t][4 * r], col.o[t][4 * r + 1], col.o[t][4 * r + 2], col.o[t][4 * r + 3]};
  barrier();
  float2 m[kPfWaves];
  float top = -__builtin_inff(), sum = 0.f;
#pragma unroll
  for (int w = 0; w < kPfWaves; ++w) {
    m[w] = ml[64 * w + lane];
    top = fmaxf(top, m[w].x);
  }
  f32x16 o = f32x16{};
#pragma unroll
  for (int w = 0; w < kPfWaves; ++w) {
    const float f = fast_exp2(m[w].x - top);
    sum += f * m[w].y;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 p = parts[((w * 4 + wave) * 4 + r) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[4 * r + e] += f * p[e];
    }
  }
  if (col.ok) store_tile<T>(a, col.row, o, 1.0f / sum, wave, h);
}

template <typename T, int G, bool F8>
hipError_t launch_typed(PrefillArgs a, bool elastic, hipStream_t st) {
  a.spread = spread_tiles((int64_t)a.batch * a.num_kv_heads, a.total_q, (int64_t)a.batch * a.max_q_len);
  constexpr int kSplitTok = kPfCols / G;
  const int64_t split = (int64_t)((a.max_q_len + kSplitTok - 1) / kSplitTok) * a.num_kv_heads * a.batch;
  // (EKV_PREFILL_SPLIT = 0 or 1 overrides, for tests and measurements)
  const char* forced = getenv("EKV_PREFILL_SPLIT");
  if (forced ? atoi(forced) != 0 : divide_units(split, (int64_t)a.max_q_len * G, a.max_len, a.len_stated != 0)) {
    const dim3 grid((unsigned)(split / a.batch), a.batch);
    if (elastic) hipLaunchKernelGGL((prefill_split_kernel<T, G, true, F8>), grid, dim3(64 * kPfWaves), 0, st, a);
    else hipLaunchKernelGGL((prefill_split_kernel<T, G, false, F8>), grid, dim3(64 * kPfWaves), 0, st, a);
    return hipGetLastError();
  }
  constexpr int kTileTok = kPfWaves * kPfCols / G;
  const int tiles = (a.max_q_len + kTileTok - 1) / kTileTok;
  const dim3 grid((unsigned)tiles * a.num_kv_heads, a.batch);
  if (elastic) hipLaunchKernelGGL((prefill_kernel<T, G, true, F8>), grid, dim3(64 * kPfWaves), 0, st, a);
  else hipLaunchKernelGGL((prefill_kernel<T, G, false, F8>), grid, dim3(64 * kPfWaves), 0, st, a);
  return hipGetLastError();
}

template <typename T, bool F8>
hipError_t launch_group(const PrefillArgs& a, int group, bool elastic, hipStream_t st) {
  switch (group) {
    case 1: return launch_typed<T, 1, F8>(a, elastic, st);
    case 2: return launch_typed<T, 2, F8>(a, elastic, st);
    case 4: return launch_typed<T, 4, F8>(a, elastic, st);
    case 8: return launch_typed<T, 8, F8>(a, elastic, st);
    case 16: return launch_typed<T, 16, F8>(a, elastic, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_prefill(const PrefillArgs& a, int dtype, int group, bool elastic, hipStream_t st) {
  if (a.batch == 0 || a.max_q_len == 0) return hipSuccess;
  if (dtype == 3) return launch_group<Fp16, true>(a, group, elastic, st);   // 8-bit pool, FP16 queries
  return dtype == 0 ? launch_group<Bf16, false>(a, group, elastic, st) : launch_group<Fp16, false>(a, group, elastic, st);
}

}  // namespace ekv
