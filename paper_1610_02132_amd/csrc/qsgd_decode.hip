// Decode kernels, fused with the sum over the K peers and the update
//   x <- x - (eta/K) sum_l Decode(M_l)          (Alg. 1, last line)
// Decode of one bucket string (Sec. 3.1, last sentences on the coding scheme):
// read the 32-bit scale, then the records; Eq. (2) turns (scale, sign, level)
// into a value.
//
// Elias codes are prefix codes: one string can only be read front to back.  The
// parallelism is across strings: every lane of a wavefront reads its own string
// (bucket g of message k), the wavefront owns gw buckets of all K messages, and
// the per-bucket offset table says where each string starts.  Records go through
// small per-string queues in LDS and are applied to an LDS accumulator such that
// every element's fp32 sum is the one taken message by message (k ascending);
// then the accumulator is streamed against x with float4 accesses.
#include <type_traits>

#include "qsgd_device.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

constexpr uint32_t kRingStride = kStrWin + 1;   // words of a lane's string ring: kStrWin and the mirror of slot 0

namespace {

// A piece of a string: words [idx, idx + kStrFetch), zeros at and past nwords; idx is a
// multiple of kStrFetch.  Strings are word-aligned, so a whole piece is one 16-byte load.
static_assert(kStrFetch == 4 && kStrWin % kStrFetch == 0, "pieces of four words");
struct __attribute__((packed, aligned(4))) StrPiece { uint32_t w[kStrFetch]; };
__device__ __forceinline__ void load_piece(const uint32_t* str, uint32_t idx, uint32_t nwords,
                                           uint32_t (&t)[kStrFetch]) {
  if (idx + kStrFetch <= nwords) {
    const StrPiece p = *reinterpret_cast<const StrPiece*>(str + idx);
#pragma unroll
    for (uint32_t j = 0; j < kStrFetch; ++j) t[j] = p.w[j];
  } else {
#pragma unroll
    for (uint32_t j = 0; j < kStrFetch; ++j) t[j] = idx + j < nwords ? str[idx + j] : 0u;
  }
}
// Stores the piece that starts at word `idx` of the string into a lane's ring (word j of the
// string in slot j % kStrWin; slot kStrWin mirrors slot 0).
__device__ __forceinline__ void ring_put_piece(uint32_t* ring, uint32_t idx,
                                               const uint32_t (&t)[kStrFetch]) {
  const uint32_t sl = idx & (kStrWin - 1u);
  uint32_t* const at = ring + sl;
#pragma unroll
  for (uint32_t j = 0; j < kStrFetch; ++j) at[j] = t[j];
  if (sl == 0) ring[kStrWin] = t[0];
}

// Entry of the Elias table for the 7-bit pattern b7 (first stream bit on top): (after, more)
// = where the bits of the LAST group after its leading 1 start, and how many they are.  The
// value of the code word is then 2^more + those bits and its length after + more + 1:
//   0......  the value 1                         (after 0, more 0)
//   1x0....  one group: 2 or 3                   (after 1, more 1)
//   1x1ab0.  two groups, the second of x+3 bits  (after 3, more x+2)
//   1x1ab1.  a third group of (second group)+1 bits follows: values 16 .. 2^16 - 1
__device__ __forceinline__ uint8_t omega_table_entry(uint32_t b7) {
  uint32_t after = 0, more = 0;
  if (b7 & 64u) {
    const uint32_t g1 = 2u | ((b7 >> 5) & 1u);
    after = 1; more = 1;
    if (b7 & 16u) {
      const uint32_t n1 = g1 + 1u;                                   // bits of the second group
      const uint32_t g2 = (b7 >> (5u - n1)) & ((1u << n1) - 1u);
      after = 3; more = n1 - 1u;
      if ((b7 >> (4u - n1)) & 1u) {                                   // the third group's leading 1
        after = 2u + n1 + 1u;
        more = g2;
      }
    }
  }
  return (uint8_t)(after | (more << 3));
}

}  // namespace

__global__ void k_decode_check(DecodeArgs a) { check_headers(a); }

// ---- fixed width: one wavefront per bucket ----------------------------------------
// Lane k < K keeps message k's scale and escape index.  A wavefront takes CH chunks
// of 256 positions at a time; for those it requests the level and sign words of
// KG messages together, so that enough bytes are in flight per wavefront, and so
// that the 128-byte lines of a message that two chunks (or the header and the
// first chunk) share are touched at one time instead of once per chunk with 15
// other messages in between (measured: the second touch came from memory again).
// The sum over the messages runs in k order in registers.
// CHECK: a field can hold a level above s (s + 1 is not a power of two).
template <int B, int CH, bool CHECK>
__global__ __launch_bounds__(256) void k_decode_fixed(DecodeArgs a) {
  if (*a.status != 0) return;
  constexpr int KG = CH >= 4 ? QSGD_FIXED_KG / 2 : QSGD_FIXED_KG;  // messages whose words are requested together
  const int lane = threadIdx.x & 63;
  const uint32_t wave_global = blockIdx.x * 4 + (threadIdx.x >> 6);
  const uint32_t wave_count = gridDim.x * 4;
  const uint32_t s = a.s, K = a.K;
  const float s_f = (float)s;
  constexpr uint32_t fmask = (1u << B) - 1u;
  constexpr int LW = B == 16 ? 2 : 1;       // level words a lane reads per message and chunk
  const uint64_t all_ok = K >= 64 ? ~0ull : ((1ull << K) - 1ull);

  for (uint32_t b = wave_global; b < a.nb; b += wave_count) {
    uint64_t base;
    uint32_t m;
    bucket_extent(a, b, base, m);
    const uint32_t lw = (m * B + 31u) >> 5, sw = (m + 31u) >> 5;
    const uint64_t str_off = (uint64_t)H_WORDS + (uint64_t)b * a.fixed_words_full;
    float my_scale = 0.f;
    uint32_t my_esc = 0xFFFFFFFFu, my_ok = 0;
    if ((uint32_t)lane < K) {
      if (str_off + 2u + lw + sw <= a.msg_words[lane]) {
        const uint32_t* str = a.msgs[lane] + str_off;
        my_scale = __uint_as_float(str[0]) / s_f;
        my_esc = str[1];
        my_ok = (my_esc == 0xFFFFFFFFu || my_esc < m) ? 1u : 0u;
      }
      if (!my_ok) { flag_corrupt(a.status); my_scale = 0.f; my_esc = 0xFFFFFFFFu; }
    }
    const uint64_t okmask = __builtin_amdgcn_ballot_w64(my_ok != 0);
    // every message is intact and every chunk of the group is complete: no per-load tests
    const bool whole = okmask == all_ok && m % (CH * kChunk) == 0;
    for (uint32_t g0 = 0; g0 < m; g0 += CH * kChunk) {
      float4 xv[CH];
      float acc[CH][4];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t e0 = g0 + (uint32_t)c * kChunk + (uint32_t)lane * 4u;
        const float* xp = a.x + base + e0;
        xv[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        acc[c][0] = acc[c][1] = acc[c][2] = acc[c][3] = 0.f;
        if (e0 + 3 < m) {
          xv[c] = load_stream(xp);
        } else if (e0 < m) {
          xv[c].x = xp[0];
          if (e0 + 1 < m) xv[c].y = xp[1];
          if (e0 + 2 < m) xv[c].z = xp[2];
        }
      }
      for (uint32_t k0 = 0; k0 < K; k0 += KG) {
        uint32_t wl[KG][CH][LW], ws[KG][CH];
        if (whole) {
#pragma unroll
          for (int t = 0; t < KG; ++t) {
            const uint32_t* lplane = a.msgs[min(k0 + t, K - 1u)] + str_off + 2;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
              const uint32_t e0 = g0 + (uint32_t)c * kChunk + (uint32_t)lane * 4u;
              const uint32_t li = (e0 * B) >> 5;
              wl[t][c][0] = lplane[li];
              if (LW == 2) wl[t][c][LW - 1] = lplane[li + 1];
              ws[t][c] = lplane[lw + (e0 >> 5)];
            }
          }
        } else {
#pragma unroll
          for (int t = 0; t < KG; ++t) {
            const uint32_t k = k0 + t;
            const bool live = k < K && ((okmask >> k) & 1ull);
            const uint32_t* lplane = live ? a.msgs[k] + str_off + 2 : nullptr;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
              const uint32_t e0 = g0 + (uint32_t)c * kChunk + (uint32_t)lane * 4u;
              const uint32_t li = (e0 * B) >> 5;
              wl[t][c][0] = 0; ws[t][c] = 0;
              if (LW == 2) wl[t][c][LW - 1] = 0;
              if (live && e0 < m) {
                wl[t][c][0] = lplane[li];
                if (LW == 2 && li + 1 < lw) wl[t][c][LW - 1] = lplane[li + 1];
                ws[t][c] = lplane[lw + (e0 >> 5)];
              }
            }
          }
        }
#pragma unroll
        for (int t = 0; t < KG; ++t) {
          const uint32_t k = k0 + t;
          if (k >= K) break;
          const float sc = __uint_as_float(lane_bcast(__float_as_uint(my_scale), (int)k));
          const uint32_t esc = lane_bcast(my_esc, (int)k);
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            const uint32_t c0 = g0 + (uint32_t)c * kChunk;       // uniform
            const uint32_t e0 = c0 + (uint32_t)lane * 4u;
            uint32_t z[4];
            if (B == 8) {
              z[0] = wl[t][c][0] & 0xFFu; z[1] = (wl[t][c][0] >> 8) & 0xFFu;
              z[2] = (wl[t][c][0] >> 16) & 0xFFu; z[3] = wl[t][c][0] >> 24;
            } else if (B == 16) {
              z[0] = wl[t][c][0] & 0xFFFFu; z[1] = wl[t][c][0] >> 16;
              z[2] = wl[t][c][LW - 1] & 0xFFFFu; z[3] = wl[t][c][LW - 1] >> 16;
            } else {
              const uint32_t w = wl[t][c][0] >> ((e0 * B) & 31u);
              z[0] = w & fmask; z[1] = (w >> B) & fmask; z[2] = (w >> (2 * B)) & fmask;
              z[3] = (w >> (3 * B)) & fmask;
            }
            float mag[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) mag[j] = sc * (float)z[j];
            // rare, wave-uniform: this message's top-level value lies in this chunk
            if (esc - c0 < kChunk) {
              const float top = sc * s_f;
#pragma unroll
              for (int j = 0; j < 4; ++j)
                if (esc == e0 + j) mag[j] = top;
            }
            if (CHECK) {
              if (max(max(z[0], z[1]), max(z[2], z[3])) > s) flag_corrupt(a.status);
            }
            const uint32_t sg = ws[t][c] >> (e0 & 31u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              // the sign bit goes into the product (-0 for a zero level adds like +0)
              acc[c][j] += __uint_as_float(((sg << (31 - j)) & 0x80000000u) | __float_as_uint(mag[j]));
            }
          }
        }
      }
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t e0 = g0 + (uint32_t)c * kChunk + (uint32_t)lane * 4u;
        float* xp = a.x + base + e0;
        float4 v = xv[c];
        if (a.step) {
          v.x = fmaf(-a.c, acc[c][0], v.x); v.y = fmaf(-a.c, acc[c][1], v.y);
          v.z = fmaf(-a.c, acc[c][2], v.z); v.w = fmaf(-a.c, acc[c][3], v.w);
        } else {
          v.x += acc[c][0]; v.y += acc[c][1]; v.z += acc[c][2]; v.w += acc[c][3];
        }
        if (e0 + 3 < m) {
          store_stream(xp, v);
        } else if (e0 < m) {
          xp[0] = v.x;
          if (e0 + 1 < m) xp[1] = v.y;
          if (e0 + 2 < m) xp[2] = v.z;
        }
      }
    }
  }
}

// ---- Elias codes: one lane per string, gw buckets x K messages per wavefront -------
// The bucket is walked in windows of `win` (<= 256) positions.  Per wavefront:
//  (1) x of a window is requested into registers well ahead of its use (at the
//      start of the window, or a whole window earlier: see kAhead);
//  (2) every lane parses ahead into its own ring of records.  Its string comes
//      through a small per-lane ring of words in LDS that is refilled in pieces
//      (a 128-byte line of a message is then fetched a few times, not once per
//      code word), and the parser itself works on a 64-bit register of unread bits;
//  (3) records are applied to an LDS accumulator, but only up to the position
//      every string has been parsed to, and such that every element's terms are
//      added in message order (see the apply step below);
//  (4) registers and accumulator are combined and stored.
// The kernel is bound by latency and instruction issue, not by bytes: small LDS
// per wavefront (short rings, 256-position windows) buys occupancy, which
// measured better than longer rings or windows.

// CODE: sparse or dense Elias code.  LG: groups a level's code word may have.
// KLOOP: apply the queued records message by message (dense messages) instead of
// counting the terms of every position first (sparse ones); see the apply step.
// Q16: queued records are 16 bits wide (s <= 4: the level, stored minus one, fits two
// bits beside 13 bits of position and the sign); the smaller rings let two more
// wavefronts live on a compute unit (c5: 2.77 -> 2.60 ms).
template <int CODE, int LG, int NQ, bool KLOOP, bool Q16>
__device__ __forceinline__ void decode_elias_body(const DecodeArgs& a, float* acc,
                                                  std::conditional_t<Q16, uint16_t, uint32_t>* queue,
                                                  uint32_t* swin, uint32_t b0, uint32_t gcount) {
  using qrec_t = std::conditional_t<Q16, uint16_t, uint32_t>;
  constexpr uint32_t kLevBias = Q16 ? 1u : 0u;
  constexpr uint32_t kRecWords = rec_words(Q16);
  constexpr bool kSparse = CODE == QSGD_CODE_SPARSE;
  // a whole record in one 32-bit peek: gap <= 21 bits, sign, level <= 7 bits
  constexpr bool kNarrow = !kSparse || LG <= 2;
  const uint32_t K = a.K, gw = a.gw, win = a.win, s = a.s;
  // ring depth: the message-by-message apply hands ring slot r of string (g, k) to lane
  // (g, r), so gw * depth <= 64 there
  constexpr bool kloop = KLOOP;
  const uint32_t rec = kloop ? a.rec : kRec;
  // ring slot idx of lane l: lane-major where other lanes read a string's slots side
  // by side (message loop), slot-major where a lane only reads its own ring
  auto qidx = [&](uint32_t l, uint32_t idx) -> uint32_t {
    return kloop ? l * rec + idx : idx * 64u + l;
  };
  constexpr uint32_t winp = kChunk;  // accumulator stride per bucket
  const int lane = threadIdx.x;
  const uint64_t pay = (uint64_t)H_WORDS + a.table_words;

  // ---- open this lane's string -----------------------------------------------------
  const uint32_t g = lane / K, k = lane - g * K;
  const uint32_t b = b0 + g;
  // The record a lane has decoded and not yet queued: (pend_pos, pend_lev, pend_neg), pend_pos
  // 1-based, kDone when there is none (the string has ended or is damaged).  One number says
  // both whether there is a record and where it falls, and the parse loop below has one
  // predicate per trip: every instruction of that loop, scalar ones included, is a step of
  // a chain that a lane's string forces to be serial.
  constexpr uint32_t kDone = 0xFFFFFFFFu;
  uint32_t m = 0;         // elements in this lane's bucket
  uint32_t endbit = 0;    // records end here
  uint32_t bitpos = 32;   // next unread bit (after the scale)
  uint32_t nwords = 0;
  uint32_t pend_pos = kDone, pend_lev = 0, pend_neg = 0;
  const uint32_t* str = nullptr;
  bool open = false;
  float my_scale = 0.f;
  if (g < gcount) {
    uint64_t base_unused;
    bucket_extent(a, b, base_unused, m);
    const uint32_t* msg = a.msgs[k];
    const uint32_t o0 = msg[H_WORDS + b], o1 = msg[H_WORDS + b + 1];
    if (o0 < o1 && pay + o1 <= a.msg_words[k]) {
      nwords = o1 - o0;
      str = msg + pay + o0;
      my_scale = __uint_as_float(str[0]) / (float)s;
      open = true;
      if (kSparse) {
        const uint32_t last = str[nwords - 1];
        endbit = nwords * 32u - 1u - (uint32_t)(__ffs((int)last) - 1);
        if (last == 0 || endbit < 32u) open = false;
      } else {
        endbit = nwords * 32u;
      }
    }
    if (!open) flag_corrupt(a.status);
  }
  if (!open) my_scale = 0.f;

  // The lane's view of its string: the last kStrWin words fetched, as a ring in LDS: word j
  // of the string in slot j % kStrWin of the lane's kStrWin + 1 slots; the last slot mirrors
  // slot 0, so that two consecutive words are always two consecutive slots (one LDS read
  // of a pair), and the odd stride keeps the lanes on distinct banks.  A string is touched
  // once per kStrFetch words instead of once per record, and the touches of one wavefront
  // happen together at the top of a round, so a 128-byte line of a message is pulled from
  // memory a few times rather than once per code word.
  uint32_t* const ring = swin + (uint32_t)lane * kRingStride;
  uint8_t* const otab = reinterpret_cast<uint8_t*>(swin + 64u * kRingStride);   // Elias table
  uint32_t sfill = 0;   // words [sfill - kStrWin, sfill) of the string are in the ring
  auto fetch = [&]() {
    uint32_t t[kStrFetch];
    load_piece(str, sfill, nwords, t);
    ring_put_piece(ring, sfill, t);
    sfill += kStrFetch;
  };
  // The 32 stream bits from bit `at` on, out of the ring (bit j of the stream is bit
  // 31 - j % 32 of word j / 32).  The parser keeps a bit position instead of a shift
  // register: the vector ALU bounds this kernel, and this way it only aligns two words.
  auto peek = [&](uint32_t at) -> uint32_t {
    const uint32_t off = at & 31u;
    const uint32_t* const pw = ring + ((at >> 5) & (kStrWin - 1u));
    const uint32_t wa = pw[0], wb = pw[1];
    const uint32_t sh = __builtin_amdgcn_alignbit(wa, wb, 32u - off);   // (off = 0 gives wb)
    return off ? sh : wa;
  };
  // Recursive Elias code (App. A.2) through a table: the entry (after, more) of the next 7
  // bits says where the last group's bits after its leading 1 start and how many they are;
  // the value is 2^more + those bits, the code word after + more + 1 bits (with its closing
  // 0, which `open_end` checks: its top bit is set if the word does not end there).
  // Values below 2^16 (three groups).
  auto omega_tab = [&](uint32_t w, uint32_t& len, uint32_t& open_end) -> uint32_t {
    const uint32_t e = otab[w >> 25];
    const uint32_t after = e & 7u, more = e >> 3;
    const uint32_t y = w << after;
    const uint32_t rest = __builtin_amdgcn_ubfe(y, 32u - more, more);   // (more = 0: 0)
    open_end = y << more;
    len = after + more + 1u;
    return (1u << more) | rest;
  };
  // The code words of 1 .. 4 ("0", "100", "110", "101000") from their first three bits, for
  // s <= 4: nibble b of the two constants is the value and the length for the top bits b
  // ("111" would be a value of 8 or more, and "101" has to go on with "000").  No table
  // look-up, that is one LDS round trip less in the chain from one record to the next.
  auto omega_small = [&](uint32_t w, uint32_t& len, uint32_t& open_end) -> uint32_t {
    const uint32_t six = w >> 26, b = six >> 3;
    len = (0x03631111u >> (4u * b)) & 0xFu;
    open_end = ((b == 7u) | ((b == 5u) & (six != 0x28u))) ? 0x80000000u : 0u;
    return (0x03421111u >> (4u * b)) & 0xFu;
  };
  // A record reads at most the two words at bitpos / 32 (kNarrow) or one more, so a lane may
  // parse while bitpos is below this limit (none once the whole string is in the ring: past
  // its end the ring may hold anything, those bits lie behind endbit).
  auto parse_limit = [&]() -> uint32_t {
    return sfill >= nwords ? 0xFFFFFFFFu : (sfill - (kNarrow ? 1u : 2u)) * 32u;
  };

  // Reads the next record into pend_*; `pos` is the position of the one before (0 at the
  // start of the string).  pend_pos = kDone at the end of the string.
  uint32_t bad = 0;   // a record that cannot be: remembered here, reported after the parse pass
  auto advance = [&](uint32_t pos) {
    uint32_t w = peek(bitpos);
    if (kSparse) {
      const bool more = bitpos < endbit;
      uint32_t gl, ll, e1, e2;
      const uint32_t gap = omega_tab(w, gl, e1);
      if (!kNarrow) w = peek(bitpos + gl); else w <<= gl;
      pend_neg = w >> 31;
      const uint32_t lev = Q16 ? omega_small(w << 1, ll, e2) : omega_tab(w << 1, ll, e2);
      bitpos += gl + 1u + ll;
      pos += gap;
      pend_lev = lev;
      // (no short cuts between the tests: as plain mask arithmetic they cost no branch)
      const bool bad_rec = ((int)(e1 | e2) < 0) | (lev > s) | (pos > m) | (bitpos > endbit);
      bad |= (more & bad_rec) ? 1u : 0u;
      pend_pos = (more & !bad_rec) ? pos : kDone;
    } else {
      const bool more = pos < m;
      uint32_t ll, e2;
      const uint32_t lev1 = omega_tab(w << 1, ll, e2);
      bitpos += 1u + ll;
      pend_neg = w >> 31;
      pend_lev = lev1 - 1u;
      const bool bad_rec = ((int)e2 < 0) | (lev1 > s + 1u) | (bitpos > endbit);
      bad |= (more & bad_rec) ? 1u : 0u;
      pend_pos = (more & !bad_rec) ? pos + 1u : kDone;
    }
  };
  // the table: entry of the 7-bit pattern b7 (first stream bit on top)
  for (uint32_t b7 = lane; b7 < 128u; b7 += 64) otab[b7] = omega_table_entry(b7);
  if (open) {
    fetch();
    fetch();
  }
  __syncthreads();
  if (open) advance(0u);
  if (bad) { flag_corrupt(a.status); bad = 0; }

  for (uint32_t j = lane; j < gw * winp; j += 64) acc[j] = 0.f;
  __syncthreads();

  // A window is at most 256 positions (winp = 256): quad q of the x registers is
  // bucket q of this wavefront, lane l holds positions 4l..4l+3 of the window.
  uint32_t qhead = 0, qcnt = 0;            // this lane's ring of queued records
  uint32_t* const accu = reinterpret_cast<uint32_t*>(acc);
  const uint32_t grow = (g < gw ? g : 0u) * winp;   // this lane's accumulator row
  const uint32_t dump = gw * winp + kRecWords + 64u * kRingStride + 32u + (uint32_t)lane;
  uint32_t* const counts = accu + gw * winp + kRecWords + 64u * kRingStride + 32u + 64u;
  uint32_t* const heads = counts + 64;
  float* const scales = reinterpret_cast<float*>(counts + 128);
  const uint32_t i = (uint32_t)lane * 4u;
  // x of one window into registers: quad qi is bucket qi of this wavefront.
  // The common case, decided per window on the scalar unit: the wavefront has all its NQ
  // buckets and the window lies inside every one of them.  Then loads and stores need no
  // per-lane bounds (the general code below costs about a hundred vector instructions per
  // window, and the vector ALU is what bounds this kernel).
  uint64_t xbase[NQ];
  uint32_t xlen_min = 0xFFFFFFFFu;
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi) {
    xbase[qi] = 0;
    uint32_t mb = 0;
    if ((uint32_t)qi < gcount) bucket_extent(a, b0 + (uint32_t)qi, xbase[qi], mb);
    xlen_min = min(xlen_min, mb);
  }
  auto whole_window = [&](uint32_t ws) -> bool { return ws + win <= xlen_min && win == kChunk; };
  auto load_x = [&](float4 (&dst)[NQ], uint32_t ws) {
    if (whole_window(ws)) {
#pragma unroll
      for (int qi = 0; qi < NQ; ++qi) dst[qi] = load_stream(a.x + xbase[qi] + ws + i);
      return;
    }
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi) {
      dst[qi] = make_float4(0.f, 0.f, 0.f, 0.f);
      if ((uint32_t)qi < gcount) {
        uint64_t base;
        uint32_t mb;
        bucket_extent(a, b0 + (uint32_t)qi, base, mb);
        const uint32_t cntw = ws < mb ? min(win, mb - ws) : 0u;
        const float* xp = a.x + base + ws + i;
        if (i + 3 < cntw) {
          dst[qi] = load_stream(xp);
        } else {
          if (i + 0 < cntw) dst[qi].x = xp[0];
          if (i + 1 < cntw) dst[qi].y = xp[1];
          if (i + 2 < cntw) dst[qi].z = xp[2];
        }
      }
    }
  };
  // Order of the memory operations (the wait counter retires them in order): the x
  // values are requested at the start of a window and used at its end; the next piece
  // of a string is requested into registers at the top of a parse round (counting apply)
  // and at the end of a window, BEFORE that window's stores, and moved into the ring at
  // the top of the following round, so that waiting for string words never waits for a
  // store, and a round's own work hides their latency and that of the x values.
  uint32_t tw[kStrFetch], tw_base = 0;   // string words on their way: [tw_base, tw_base + kStrFetch)
  bool tw_pending = false;
  auto commit_pending = [&]() {
    if (tw_pending && sfill == tw_base) {   // (a fetch on demand may have overtaken them)
      ring_put_piece(ring, sfill, tw);
      sfill += kStrFetch;
    }
    tw_pending = false;
  };
  // Requests the next piece of the string into registers; commit_pending() moves it
  // into the ring later, so the round in between hides the latency.
  auto request_next = [&]() {
    tw_pending = pend_pos != kDone && sfill < nwords && sfill - (bitpos >> 5) <= kStrWin - kStrFetch;
    tw_base = sfill;
    if (tw_pending) load_piece(str, sfill, nwords, tw);
  };
  // Message-by-message apply: x is requested a whole window ahead, because its rounds
  // wait for string words at once and would wait for x with them.  Counting apply: the
  // string words of a round arrive a round later, so x is requested at the start of its
  // own window and one register set is enough (one more wavefront per SIMD).
  constexpr bool kAhead = KLOOP;
  float4 xr[NQ], xn[NQ];
  if constexpr (kAhead) load_x(xr, 0);
  for (uint32_t ws = 0; ws < a.d; ws += win) {
    const uint32_t wend = ws + win;  // positions (1-based) up to wend fall in this window
    if constexpr (kAhead) {
      if (wend < a.d) load_x(xn, wend);
    } else {
      load_x(xr, ws);
    }
    // ---- rounds: parse ahead into the rings, apply what is due --------------------------
    // A position may only be applied once EVERY string has been parsed past it,
    // or an element could receive message 5's term before message 2's.  `limit`
    // is the smallest position still pending in any string, minus 1, capped at
    // the window end; queued records past it wait in the ring.  Parsing is lazy:
    // nobody parses while every string is already past the window end, and when
    // some string is not, all of them fill their rings (fewer, fuller passes of
    // the divergent parse loop).
    for (;;) {
      // A parse pass costs as many trips of the divergent loop as its busiest lane
      // takes, so passes are short and start when most lanes can use all the trips
      // (their rings have room), or when a lane is out of records for this window.
      const uint64_t needy = __builtin_amdgcn_ballot_w64(pend_pos <= wend);
      const uint32_t nroom = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(pend_pos != kDone && qcnt + kRoom <= rec));
      if (needy != 0 || nroom >= kParseLanes) {
        // top up the string rings together, then parse
        commit_pending();
        if constexpr (KLOOP) {
          // dense strings use up a piece in a round or two: have it now
          if (pend_pos != kDone && sfill < nwords && sfill - (bitpos >> 5) <= kStrWin - kStrFetch) fetch();
        } else {
          request_next();   // arrives while this round parses and applies
        }
        const uint32_t trips = __popcll(needy) >= 32 ? rec : kParse;   // dense data: no imbalance
        const uint32_t plim = parse_limit();
        for (uint32_t np = 0; np < trips; ++np) {
          const bool c1 = pend_pos != kDone, c2 = qcnt < rec, c3 = bitpos < plim;
          const bool act = c1 & c2 & c3;
          // (the wavefront's vote from the three comparisons' own masks: a vote on their
          // conjunction first turns it into a register and compares again)
          if ((__builtin_amdgcn_ballot_w64(c1) & __builtin_amdgcn_ballot_w64(c2) &
               __builtin_amdgcn_ballot_w64(c3)) == 0)
            break;
          if (act) {
            if (kSparse || pend_lev) {   // (Code_s records always carry a level >= 1)
              queue[qidx((uint32_t)lane, (qhead + qcnt) & (rec - 1))] =
                  (qrec_t)((pend_pos - 1u) | (pend_neg << 13) | ((pend_lev - kLevBias) << 14));
              ++qcnt;
            }
            advance(pend_pos);
          }
        }
        if (bad) { flag_corrupt(a.status); bad = 0; }
      }
      if constexpr (KLOOP) {
        // Dense data: nearly every ring slot is due in every round, so the records are
        // applied message by message: in turn kk, lane (g2, r) takes slot r of string
        // (g2, kk), and all strings of one message run side by side.
        uint32_t limit = wave_min_u32(pend_pos - 1u);   // (kDone - 1: no limit from this lane)
        limit = min(limit, wend);   // 0-based positions below `limit` are due
        counts[lane] = qcnt;
        heads[lane] = qhead;
        scales[lane] = my_scale;
        __syncthreads();
        const uint32_t g2 = (uint32_t)lane / rec, r = (uint32_t)lane - g2 * rec;
        for (uint32_t kk = 0; kk < K; ++kk) {
          if (g2 < gw) {
            const uint32_t sl = g2 * K + kk;
            if (r < counts[sl]) {
              const uint32_t q = queue[qidx(sl, (heads[sl] + r) & (rec - 1))];
              const uint32_t p0 = q & 0x1FFFu;
              if (p0 < limit) {
                const float mag = scales[sl] * (float)((q >> 14) + kLevBias);
                acc[g2 * winp + ((p0 - ws) & (winp - 1u))] += ((q >> 13) & 1u) ? -mag : mag;
              }
            }
          }
          __syncthreads();
        }
        // drop what was applied from the front of the ring
        while (qcnt && (queue[qidx((uint32_t)lane, qhead)] & 0x1FFFu) < limit) {
          qhead = (qhead + 1u) & (rec - 1);
          --qcnt;
        }
        if (limit == wend) break;
        continue;
      }
      // At most kApply records per lane are applied in a round: a lane that holds
      // more caps the limit at its first record beyond them.
      uint32_t qv[kApply + 1], ad[kApply];
#pragma unroll
      for (uint32_t t = 0; t <= kApply; ++t)
        qv[t] = queue[((qhead + t) & (kRec - 1)) * 64u + lane];
      const uint32_t cap = qcnt > kApply ? (qv[kApply] & 0x1FFFu) : 0xFFFFFFFFu;
      uint32_t limit = wave_min_u32(min(pend_pos - 1u, cap));   // (kDone - 1: no limit)
      limit = min(limit, wend);   // 0-based positions below `limit` are due
      // ---- apply the due records of this lane's own ring ---------------------------------
      // All records of one position become due in the same round, and the position's word of
      // the accumulator is 0 until then.  That word first collects WHO has a term there, a bit
      // per message (K <= 32 on this path): a record's rank among the set bits below its own is
      // its turn in the sum that Alg. 1's last line takes message by message.  Then
      //   turn 0    stores its term (0 + t = t),
      //   turn r    adds its term to what turns 0 .. r-1 left, r = 1, 2, ... while any lane
      //             still has a record waiting: as many passes as the busiest position of
      //             the round has terms, not one per message.
      // Every pass handles the ring entries in groups of kGrp with straight-line code: entries
      // that do not take part read and write the lane's dump word instead of branching, so
      // that the LDS operations of a group are in flight together.
      constexpr uint32_t kGrp = 4;
      {
        // (positions ascend along a string, so the due entries are the first `ndue` of the ring)
        bool due[kApply];
        uint32_t ndue = 0;
#pragma unroll
        for (uint32_t t = 0; t < kApply; ++t) {
          const uint32_t p0 = qv[t] & 0x1FFFu;
          ad[t] = grow + ((p0 - ws) & (winp - 1u));
          due[t] = (t < qcnt) & (p0 < limit);
          ndue += due[t] ? 1u : 0u;
        }
        // uniform: does any lane apply an entry of the group that starts at t0?  (a vote per
        // group costs a comparison; the wavefront's maximum would cost a dozen shuffles)
        bool grp[kApply / kGrp];
#pragma unroll
        for (uint32_t t0 = 0; t0 < kApply; t0 += kGrp)
          grp[t0 / kGrp] = __builtin_amdgcn_ballot_w64(ndue > t0) != 0;
        const uint32_t kbit = 1u << k;
#pragma unroll
        for (uint32_t t0 = 0; t0 < kApply; t0 += kGrp) {
          if (!grp[t0 / kGrp]) break;
#pragma unroll
          for (uint32_t j = 0; j < kGrp; ++j) atomicOr(&accu[ad[t0 + j]], due[t0 + j] ? kbit : 0u);
        }
        __syncthreads();
        // a byte per ring entry: its turn, 0xFF for an entry that is not due
        uint32_t turn[kApply / 4];
        static_assert(kApply % 4 == 0, "turns are packed four to a word");
#pragma unroll
        for (uint32_t t = 0; t < kApply / 4; ++t) turn[t] = 0xFFFFFFFFu;
        uint32_t last = 0;   // the highest turn of this lane's entries
#pragma unroll
        for (uint32_t t0 = 0; t0 < kApply; t0 += kGrp) {
          if (!grp[t0 / kGrp]) break;
          uint32_t who[kGrp];
#pragma unroll
          for (uint32_t j = 0; j < kGrp; ++j) who[j] = accu[ad[t0 + j]];
#pragma unroll
          for (uint32_t j = 0; j < kGrp; ++j) {
            const uint32_t t = t0 + j;
            const uint32_t mine = (uint32_t)__popc(who[j] & (kbit - 1u));
            const uint32_t sh = 8u * (t & 3u);
            turn[t / 4] = due[t] ? (turn[t / 4] & ~(0xFFu << sh)) | (mine << sh) : turn[t / 4];
            last = due[t] ? max(last, mine) : last;
          }
        }
        __syncthreads();
        float term[kApply];
#pragma unroll
        for (uint32_t t = 0; t < kApply; ++t) {
          const float mag = my_scale * (float)((qv[t] >> 14) + kLevBias);
          term[t] = ((qv[t] >> 13) & 1u) ? -mag : mag;
        }
#pragma unroll
        for (uint32_t t0 = 0; t0 < kApply; t0 += kGrp) {
          if (!grp[t0 / kGrp]) break;
#pragma unroll
          for (uint32_t j = 0; j < kGrp; ++j) {
            const uint32_t t = t0 + j;
            const bool now = ((turn[t / 4] >> (8u * (t & 3u))) & 0xFFu) == 0u;
            acc[now ? ad[t] : dump] = term[t];
          }
        }
        __syncthreads();
        for (uint32_t r = 1; __builtin_amdgcn_ballot_w64(last >= r) != 0; ++r) {
#pragma unroll
          for (uint32_t t0 = 0; t0 < kApply; t0 += kGrp) {
            if (!grp[t0 / kGrp]) break;
            float old[kGrp];
            uint32_t at[kGrp];
#pragma unroll
            for (uint32_t j = 0; j < kGrp; ++j) {
              const uint32_t t = t0 + j;
              const bool now = ((turn[t / 4] >> (8u * (t & 3u))) & 0xFFu) == r;
              at[j] = now ? ad[t] : dump;
              old[j] = acc[at[j]];
            }
#pragma unroll
            for (uint32_t j = 0; j < kGrp; ++j) acc[at[j]] = old[j] + term[t0 + j];
          }
          __syncthreads();
        }
        qhead = (qhead + ndue) & (kRec - 1);
        qcnt -= ndue;
        if (limit == wend) break;   // uniform: every string is parsed past this window
      }
    }
    // ---- string words requested a window ago arrive; request the next ones ---------------
    commit_pending();
    request_next();
    // ---- combine the accumulator with x and store ------------------------------------
    if (whole_window(ws)) {
#pragma unroll
      for (int qi = 0; qi < NQ; ++qi) {
        float* ap = acc + qi * winp + i;
        const float4 av = *reinterpret_cast<float4*>(ap);
        *reinterpret_cast<float4*>(ap) = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 xv = xr[qi];
        if (a.step) {
          xv.x = fmaf(-a.c, av.x, xv.x); xv.y = fmaf(-a.c, av.y, xv.y);
          xv.z = fmaf(-a.c, av.z, xv.z); xv.w = fmaf(-a.c, av.w, xv.w);
        } else {
          xv.x += av.x; xv.y += av.y; xv.z += av.z; xv.w += av.w;
        }
        store_stream(a.x + xbase[qi] + ws + i, xv);
      }
    } else {
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi) {
      if ((uint32_t)qi < gcount) {
        uint64_t base;
        uint32_t mb;
        bucket_extent(a, b0 + (uint32_t)qi, base, mb);
        const uint32_t cntw = ws < mb ? min(win, mb - ws) : 0u;
        float* xp = a.x + base + ws + i;
        float* ap = acc + qi * winp + i;
        if (i < cntw) {
          const float4 av = *reinterpret_cast<float4*>(ap);
          *reinterpret_cast<float4*>(ap) = make_float4(0.f, 0.f, 0.f, 0.f);
          float4 xv = xr[qi];
          if (a.step) {
            xv.x = fmaf(-a.c, av.x, xv.x); xv.y = fmaf(-a.c, av.y, xv.y);
            xv.z = fmaf(-a.c, av.z, xv.z); xv.w = fmaf(-a.c, av.w, xv.w);
          } else {
            xv.x += av.x; xv.y += av.y; xv.z += av.z; xv.w += av.w;
          }
          if (i + 3 < cntw) {
            store_stream(xp, xv);
          } else {
            xp[0] = xv.x;
            if (i + 1 < cntw) xp[1] = xv.y;
            if (i + 2 < cntw) xp[2] = xv.z;
          }
        }
      }
    }
    }
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi)
      if constexpr (kAhead) xr[qi] = xn[qi];
    __syncthreads();
  }
}

template <int CODE, int LG, int NQ, bool KLOOP, bool Q16>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NQ == 4 && !KLOOP ? QSGD_DEC_WAVES : 1)))
void k_decode_elias(DecodeArgs a) {
  if (*a.status != 0) return;
  extern __shared__ uint32_t smem[];
  // LDS: [acc: gw*winp floats][record rings][string rings: 64*kRingStride][Elias table: 32][dump 64]
  //      [counts 64][heads 64][scales 64]
  using qrec_t = std::conditional_t<Q16, uint16_t, uint32_t>;
  const uint32_t gw = a.gw, winp = a.winp;
  float* const acc = reinterpret_cast<float*>(smem);
  qrec_t* const queue = reinterpret_cast<qrec_t*>(smem + gw * winp);
  uint32_t* const swin = smem + gw * winp + rec_words(Q16);
  const uint32_t b0 = blockIdx.x * gw;
  const uint32_t gcount = min(gw, a.nb - b0);  // buckets this wavefront really has
  decode_elias_body<CODE, LG, NQ, KLOOP, Q16>(a, acc, queue, swin, b0, gcount);
}

hipError_t launch_decode_check(const DecodeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_decode_check, dim3(1), dim3(64), 0, st, a);
  return hipGetLastError();
}

template <int CH, bool CHECK>
static void launch_fixed_ch(const DecodeArgs& a, dim3 grid, dim3 block, hipStream_t st) {
  switch (a.fixed_bits) {
    case 2: hipLaunchKernelGGL((k_decode_fixed<2, CH, CHECK>), grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_decode_fixed<4, CH, CHECK>), grid, block, 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_decode_fixed<8, CH, CHECK>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((k_decode_fixed<16, CH, CHECK>), grid, block, 0, st, a); break;
  }
}

template <bool CHECK>
static void launch_fixed_check(const DecodeArgs& a, dim3 grid, dim3 block, hipStream_t st) {
  if (a.d <= kChunk) launch_fixed_ch<1, CHECK>(a, grid, block, st);
  else if (a.d <= 2 * kChunk) launch_fixed_ch<2, CHECK>(a, grid, block, st);
  else launch_fixed_ch<4, CHECK>(a, grid, block, st);
}

hipError_t launch_decode_fixed(const DecodeArgs& a, uint32_t blocks, hipStream_t st) {
  const dim3 grid(blocks), block(256);
  const bool check = ((1ull << a.fixed_bits) - 1ull) > a.s;
  if (check) launch_fixed_check<true>(a, grid, block, st);
  else launch_fixed_check<false>(a, grid, block, st);
  return hipGetLastError();
}

template <int CODE, int NQ, bool KLOOP>
static hipError_t launch_elias_kl(const DecodeArgs& a, int lg, uint32_t blocks, size_t lds,
                                  hipStream_t st) {
  const dim3 grid(blocks), block(64);
  if constexpr (CODE == QSGD_CODE_SPARSE && !KLOOP) {
    if (a.q16) {  // s <= 4: one or two groups
      if (lg == 1) hipLaunchKernelGGL((k_decode_elias<CODE, 1, NQ, false, true>), grid, block, lds, st, a);
      else hipLaunchKernelGGL((k_decode_elias<CODE, 2, NQ, false, true>), grid, block, lds, st, a);
      return hipGetLastError();
    }
  }
  switch (lg) {
    case 1: hipLaunchKernelGGL((k_decode_elias<CODE, 1, NQ, KLOOP, false>), grid, block, lds, st, a); break;
    case 2: hipLaunchKernelGGL((k_decode_elias<CODE, 2, NQ, KLOOP, false>), grid, block, lds, st, a); break;
    case 3: hipLaunchKernelGGL((k_decode_elias<CODE, 3, NQ, KLOOP, false>), grid, block, lds, st, a); break;
    default: hipLaunchKernelGGL((k_decode_elias<CODE, 4, NQ, KLOOP, false>), grid, block, lds, st, a); break;
  }
  return hipGetLastError();
}

template <int CODE, int NQ>
static hipError_t launch_elias_nq(const DecodeArgs& a, int lg, uint32_t blocks, size_t lds,
                                  hipStream_t st) {
  return a.kloop ? launch_elias_kl<CODE, NQ, true>(a, lg, blocks, lds, st)
                 : launch_elias_kl<CODE, NQ, false>(a, lg, blocks, lds, st);
}

template <int CODE>
static hipError_t launch_elias_code(const DecodeArgs& a, int lg, uint32_t blocks, size_t lds,
                                    hipStream_t st) {
  const uint32_t nq = a.gw;  // float4 of x per lane per window: one per bucket
  if (nq <= 4) return launch_elias_nq<CODE, 4>(a, lg, blocks, lds, st);
  if (nq <= 8) return launch_elias_nq<CODE, 8>(a, lg, blocks, lds, st);
  return launch_elias_nq<CODE, 16>(a, lg, blocks, lds, st);
}

// Groups in the longest level code word: Elias(s) (sparse) or Elias(s + 1) (dense).
hipError_t launch_decode_elias(const DecodeArgs& a, uint32_t blocks, size_t lds, hipStream_t st) {
  const uint32_t top = a.code == QSGD_CODE_SPARSE ? a.s : a.s + 1u;
  const int lg = top <= 3 ? 1 : top <= 15 ? 2 : top <= 65535 ? 3 : 4;
  if (a.code == QSGD_CODE_SPARSE) return launch_elias_code<QSGD_CODE_SPARSE>(a, lg, blocks, lds, st);
  return launch_elias_code<QSGD_CODE_DENSE>(a, lg, blocks, lds, st);
}

}  // namespace qsgd
