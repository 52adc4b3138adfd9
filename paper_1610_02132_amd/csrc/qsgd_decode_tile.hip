// Elias codes, dense strings: a tile of signed levels, summed in registers.
//
// Where most coordinates carry a nonzero level (Code'_s, or Code_s with s^2 of the order of
// d: Lemma 3.1 (iii)), a window of kTileW positions holds about as many records per string
// as positions, and every position receives up to K terms whose fp32 sum has to be taken in
// message order.  So the two halves of the work are separated by the data layout:
//   phase 1  every lane reads its own string (bucket g of message k) up to the end of the
//            window and writes signed levels as bytes into its own row of a tile in LDS
//            (64 rows, zero = no record): plain stores, no two lanes share a byte.
//   phase 2  lane l owns positions 4 (l % 32) .. + 3 of the window in every second bucket:
//            it reads its four bytes of the rows (g, 0) .. (g, K-1) in message order, turns
//            them into scale_k * level and adds them up in registers: the sum
//            ((0 + g^0) + g^1) + ... of Alg. 1's last line by construction, then the update
//            of x (requested at the start of the window).
// Levels must fit a signed byte (s <= 127).
//
// Phase 1 is bound by the chain of dependent instructions and LDS round trips that a prefix
// code forces from one record to the next (a wavefront issues a dependent instruction every 8
// to 10 clocks), so it takes several records per step: the next kTabBits bits of the string
// index a table in LDS whose entry says which levels the next four positions get, how many
// positions are decided and how many bits were used.  For Code_s an entry may end behind a
// gap whose sign and level do not fit any more; the second half of the table continues from
// there.  kLooks look-ups are made per 32 bits taken from the string.  What the table does
// not hold (code words longer than an entry, levels above s, anything malformed) has an entry
// of length 0 and takes the general reader, one token at a time.  Behind the string's end the
// lane sees ones, which complete no code word, so no record is ever made up from padding.
//
// Measured (step over K messages; before: one record per trip, two look-ups for gap and level
// and about 40 instructions in a row, a workgroup per wavefront):
//   25.6M values, s = 16, d = 512, Code_s, K = 8     301 -> 110 us
//   25.6M values, s = 16, d = 512, Code'_s, K = 4    240 ->  81 us
// Table of 2^9 / 2^10 / 2^11 entries with 3 / 3 / 2 look-ups: 111 / 110 / 142 us on the first
// (2^11 leaves LDS for 11 wavefronts per compute unit instead of 13: its 6250 groups of
// buckets then take three rounds instead of two).  Bytes and operations put the floor of the
// first at 45 us (HBM); the chain of phase 1 bounds it (9.5 vector and 4.2 scalar instructions per
// value and message, 0.48 vector instructions per SIMD and four clocks).
#include "qsgd_device.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

namespace {

constexpr uint32_t kTabBits = 10;
constexpr uint32_t kTabSize = 1u << kTabBits;
constexpr uint32_t kLooks = 32 / kTabBits;     // look-ups per 32 bits
// Entry, second word: bits used (0..4), largest level (8..11), state behind the entry as a byte
// offset into the table (14), positions decided (16..).  First word: see put_entry.
constexpr uint32_t kTabLen = 0x1Fu, kTabState = kTabSize * 8u;
constexpr uint32_t kTabTopShift = 8, kTabAdvShift = 16;
static_assert(kTabState >= 0x1000u && kTabState < 0x10000u, "state bit");

struct TabEntry { uint32_t x, y; };
template <int CODE> constexpr uint32_t tab_entries() { return CODE == QSGD_CODE_SPARSE ? 2 * kTabSize : kTabSize; }

constexpr TabEntry tab_entry(int code, uint32_t state, uint32_t bits) {
  const bool sparse = code == QSGD_CODE_SPARSE;
  uint32_t used = 0, pos = 0, x = 0, st = state, top = 0, recs = 0;
  for (;;) {
    const uint32_t left = kTabBits - used;
    const uint32_t rest = bits & ((1u << left) - 1u);
    if (sparse && st == 0) {
      const Token t = omega_of(rest, left);
      if (t.len == 0) break;
      used += t.len; pos += t.value - 1; st = 1;
    }
    const uint32_t room = kTabBits - used;
    if (pos >= 4 || (sparse && recs == 2) || room < 2) break;
    const uint32_t tail = bits & ((1u << room) - 1u);
    const Token t = omega_of(tail & ((1u << (room - 1)) - 1u), room - 1);   // behind the sign
    if (t.len == 0) break;
    const uint32_t neg = (tail >> (room - 1)) & 1u;
    const uint32_t lev = sparse ? t.value : t.value - 1;
    const uint32_t byte = (neg ? 0u - lev : lev) & 0xFFu;
    if (sparse) {
      // (a single record is stored twice, no record as a zero at the cursor)
      x = recs == 0 ? byte * 0x00010001u | pos * 0x01000100u : (x & 0xFFFFu) | byte << 16 | pos << 24;
    } else {
      x |= byte << (8 * pos);
    }
    used += 1 + t.len; pos += 1; recs += 1;
    if (lev > top) top = lev;
    st = 0;
  }
  return {x, used | (top << kTabTopShift) | (st ? kTabState : 0u) | (pos << kTabAdvShift)};
}

template <int CODE>
struct alignas(16) Table {
  TabEntry e[tab_entries<CODE>()];
  constexpr Table() : e() {
    for (uint32_t i = 0; i < tab_entries<CODE>(); ++i) e[i] = tab_entry(CODE, i / kTabSize, i % kTabSize);
  }
};
__device__ const Table<QSGD_CODE_SPARSE> g_table_sparse;
__device__ const Table<QSGD_CODE_DENSE> g_table_dense;

// ---- LDS of one wavefront: tile, string rings, scales ---------------------------------
constexpr uint32_t kTileW = 128;               // positions of a window
constexpr uint32_t kRowBytes = kTileW + 4;     // 33 words: the rows start on distinct banks
constexpr uint32_t kTileBytes = 64 * kRowBytes;
constexpr uint32_t kStrRing = 8;               // words of a string a lane keeps
constexpr uint32_t kPiece = 4;                 // words fetched at a time
constexpr uint32_t kRingSlots = kStrRing + 1;
constexpr uint32_t kWaveBytes = kTileBytes + 4 * 64 * kRingSlots + 4 * 64;
static_assert(kWaveBytes % 16 == 0 && kRowBytes % 4 == 0 && kTileBytes % 16 == 0, "alignment");
constexpr uint32_t kFlagBytes = 16;            // behind the wavefronts' parts: one word for all of them
constexpr uint32_t kSteps = 4;                 // steps between two top-ups of the string rings
constexpr uint32_t kDoneFlag = 0x40000000u;    // added to a finished lane's cursor
constexpr uint32_t kDone = kDoneFlag / 2;      // cursors above: finished (a cursor moves back by d at most)

struct __attribute__((packed, aligned(4))) Words4 { uint32_t w[4]; };
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// LDS by its byte address: a cursor is one register then, without a base to add.
#define QSGD_LDS __attribute__((address_space(3)))
template <typename T> __device__ __forceinline__ QSGD_LDS T* lds_at(uint32_t at) { return (QSGD_LDS T*)(uintptr_t)at; }
__device__ __forceinline__ uint32_t lds_address(void* p) { return (uint32_t)(uintptr_t)(QSGD_LDS void*)p; }

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

// A workgroup's wavefronts share the table and nothing else; each takes groups of gw
// buckets, gw * K <= 64 (lane = (bucket g, message k)), until none is left.
template <int CODE, int NP>
__global__ __launch_bounds__(64 * kTileMaxWaves) void k_decode_tile(DecodeArgs a) {
  constexpr bool kSparse = CODE == QSGD_CODE_SPARSE;
  constexpr uint32_t kEntries = tab_entries<CODE>();
  __shared__ uint4 table[kEntries / 2];
  const uint32_t status = *a.status;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];   // per wavefront: tile, string rings, scales; a word
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const uint32_t waves = blockDim.x >> 6;
  const uint32_t tab = lds_address(table);
  const uint32_t tile = lds_address(lds) + wave * kWaveBytes;
  QSGD_LDS uint32_t* const damaged = lds_at<uint32_t>(lds_address(lds) + waves * kWaveBytes);
  const uint32_t scales = tile + kTileBytes + 4u * 64u * kRingSlots;
  const uint32_t K = a.K, gw = a.gw, s = a.s;
  const uint32_t K4 = K < 4u ? K : (K + 3u) & ~3u;   // stride of a bucket's scales
  const uint64_t pay = (uint64_t)H_WORDS + a.table_words;

  const uint32_t row = tile + (uint32_t)lane * kRowBytes;
  const uint32_t ring = tile + kTileBytes + (uint32_t)lane * (4u * kRingSlots);
  const uint32_t g = (uint32_t)lane / K, k = (uint32_t)lane - g * K;
  const uint32_t half = (uint32_t)lane >> 5, i4 = ((uint32_t)lane & 31u) * 4u;
  const uint32_t tasks = (a.nb + gw - 1) / gw;
  const uint32_t* const msg = a.msgs[g < gw ? k : 0u];
  const uint64_t msg_words = a.msg_words[g < gw ? k : 0u];
  const bool has_table = msg_words >= pay;   // (whatever the header check found: asked before its word is known)

  // this lane's entry of the offset table and extent of its bucket, one group ahead
  uint32_t n_o0 = 0, n_o1 = 0, n_base = 0, n_m = 0;
  auto request_task = [&](uint32_t task) {
    n_o0 = n_o1 = n_base = n_m = 0;
    const uint32_t b = task * gw + g;
    if (task < tasks && g < gw && b < a.nb && has_table) {
      uint64_t base;
      bucket_extent(a, b, base, n_m);
      n_base = (uint32_t)base;              // (n < 2^32)
      n_o0 = msg[H_WORDS + b];
      n_o1 = msg[H_WORDS + b + 1];
    }
  };
  uint32_t task = blockIdx.x * waves + wave;
  request_task(task);

  {
    // two entries per load, eight loads in flight; a level above s is for the general reader
    // to refuse (entry of length 0)
    const uint4* src;
    if constexpr (kSparse) src = reinterpret_cast<const uint4*>(g_table_sparse.e);
    else src = reinterpret_cast<const uint4*>(g_table_dense.e);
    constexpr uint32_t kPairs = kEntries / 2;
    for (uint32_t i0 = tid; i0 < kPairs; i0 += 8u * blockDim.x) {
      uint4 v[8];
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) v[j] = src[min(i0 + j * blockDim.x, kPairs - 1u)];
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) {
        const uint32_t i = i0 + j * blockDim.x;
        const uint32_t none = i >= kTabSize / 2 ? kTabState : 0u;
        if (((v[j].y >> kTabTopShift) & 0xFu) > s) { v[j].x = 0; v[j].y = none; }
        if (((v[j].w >> kTabTopShift) & 0xFu) > s) { v[j].z = 0; v[j].w = none; }
        if (i < kPairs) table[i] = v[j];
      }
    }
    for (uint32_t j = lane; j < kTileBytes / 4u; j += kWave) *lds_at<uint32_t>(tile + 4u * j) = 0u;
    if (tid == 0) *damaged = status;
  }
  // Other workgroups set the status word meanwhile: the wavefronts go by what the first one
  // read, since a part of the table would be missing without one of them.
  __syncthreads();
  if (*damaged) return;

  for (; task < tasks; task += gridDim.x * waves) {
    const uint32_t gcount = min(gw, a.nb - task * gw);
    // ---- open this lane's string -------------------------------------------------------
    const uint32_t o0 = n_o0, o1 = n_o1, base32 = n_base, m = n_m;
    request_task(task + gridDim.x * waves);
    bool open = o0 < o1 && pay + o1 <= msg_words;
    if (g < gcount && !open) flag_corrupt(a.status);
    uint32_t nwords = open ? o1 - o0 : 0u;
    const uint32_t* const str = msg + (open ? pay + o0 : 0u);
    uint32_t first = 0, last = 1;
    if (open) { first = str[0]; last = str[nwords - 1]; }

    // The string's words come through a ring: word j in slot 7 - j % 8 behind one slot that
    // mirrors slot 7, so that words j + 1 and j are always two consecutive slots (one LDS
    // read of a pair).  np = ~(bit position - 1) counts down: its bits 5..7 are the slot and
    // its low bits the shift that aligns the pair.  Words at and past the end are ones.
    uint32_t sfill = 0, np = ~31u, endbit = 0;
    auto load_piece = [&](uint32_t at, uint32_t (&t)[kPiece]) {
      if (at + kPiece <= nwords) {
        const Words4 p = *reinterpret_cast<const Words4*>(str + at);
#pragma unroll
        for (uint32_t j = 0; j < kPiece; ++j) t[j] = p.w[j];
      } else {
#pragma unroll
        for (uint32_t j = 0; j < kPiece; ++j) t[j] = at + j < nwords ? str[at + j] : 0u;
      }
    };
    auto put_piece = [&](uint32_t (&t)[kPiece]) {
      if ((sfill + kPiece) * 32u > endbit) {
#pragma unroll
        for (uint32_t j = 0; j < kPiece; ++j) {
          const uint32_t at = (sfill + j) * 32u;
          if (at + 32u > endbit) t[j] |= at >= endbit ? 0xFFFFFFFFu : 0xFFFFFFFFu >> (endbit - at);
        }
      }
      const bool top = (sfill & kPiece) == 0;
      QSGD_LDS uint32_t* const at = lds_at<uint32_t>(ring + (top ? 4u * (kPiece + 1u) : 4u));
#pragma unroll
      for (uint32_t j = 0; j < kPiece; ++j) at[kPiece - 1u - j] = t[j];
      if (top) *lds_at<uint32_t>(ring) = t[0];
      sfill += kPiece;
    };
    auto peek = [&]() -> uint32_t {
      QSGD_LDS const uint32_t* const p = lds_at<uint32_t>(ring + 4u * ((np >> 5) & (kStrRing - 1u)));
      const uint32_t lo = p[0], hi = p[1];
      return __builtin_amdgcn_alignbit(hi, lo, np);
    };
    // a lane's cursor: LDS address, in its row, of the next undecided position
    uint32_t cur = row;
    uint32_t st = 0;          // 0, or kTabState: a gap has been read, sign and level come next
    uint32_t bad = 0;
    uint32_t tw[kPiece];
    bool tw_pending = false;
    {
      uint32_t t0[kPiece];
      load_piece(0, t0);
      load_piece(kPiece, tw);
      endbit = nwords * 32u;
      if (kSparse) {
        endbit -= 1u + (uint32_t)(__ffs((int)last) - 1);
        if (open && (last == 0 || endbit < 32u)) { open = false; flag_corrupt(a.status); }
      }
      put_piece(t0);
      put_piece(tw);
    }
    const uint32_t np_end = 0u - endbit;   // ~(endbit - 1)
    if (!open || (kSparse && np == np_end)) cur += kDoneFlag;
    const float my_scale = open ? __uint_as_float(first) / (float)s : 0.f;
    if (g < gw) *lds_at<float>(scales + 4u * (g * K4 + k)) = my_scale;
    // Where a scale is not finite, a coordinate without a record must not get 0 * scale (with
    // d % 4 != 0 in either code, as in the general path's sum of records).
    const bool records_only = (kSparse || a.d % 4u != 0) &&
        __builtin_amdgcn_ballot_w64(!(fabsf(my_scale) <= 3.402823466e+38f)) != 0;
    // windows that lie inside every one of gw buckets need no bounds
    const uint32_t m_min = gcount == gw ? wave_min_u32(g < gw ? m : 0xFFFFFFFFu) : 0u;

    // What an entry decides goes into the row.  Code_s: up to two records, (level, distance)
    // in the low and in the high half of x, two byte stores.  Code'_s: the next positions'
    // levels, joined to `part`, the bytes decided before in the cursor's word; the word is
    // stored whenever it grows.  (One unaligned 4-byte store instead costs 59 clocks: the
    // LDS takes its lanes one by one.)
    uint32_t part = 0;
    auto put_entry = [&](v2u e) {
      if constexpr (kSparse) {
        *lds_at<uint8_t>(cur + ((e.x >> 8) & 0xFFu)) = (uint8_t)e.x;
        *lds_at<uint8_t>(cur + (e.x >> 24)) = (uint8_t)(e.x >> 16);
        cur += e.y >> kTabAdvShift;
      } else {
        const uint64_t v = (uint64_t)e.x << ((cur << 3) & 24u);
        const uint32_t lo = part | (uint32_t)v;
        *lds_at<uint32_t>(cur & ~3u) = lo;
        const uint32_t next = cur + (e.y >> kTabAdvShift);
        part = (next ^ cur) < 4u ? lo : (uint32_t)(v >> 32);
        cur = next;
      }
      np -= e.y & kTabLen;
      if (kSparse) st = e.y & kTabState;
    };

    for (uint32_t ws = 0; ws < a.d; ws += kTileW) {
      // ---- x of the window's first buckets ---------------------------------------------
      float4 xr[NP];
      const bool whole = ws + kTileW <= m_min;
      auto load_x = [&](uint32_t g0) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const uint32_t gg = g0 + 2u * q + half;
          const uint32_t src = (gg * K) & 63u;      // a lane of the bucket
          const uint32_t base = (uint32_t)__shfl((int)base32, (int)src, kWave);
          const uint32_t e = ws + i4;
          const float* xp = a.x + ((uint64_t)base + e);
          if (whole && gw >= 2u * NP) {
            const v4f_any v = __builtin_nontemporal_load(reinterpret_cast<const v4f_any*>(xp));
            xr[q] = make_float4(v.x, v.y, v.z, v.w);
          } else {
            const uint32_t mb = (uint32_t)__shfl((int)m, (int)src, kWave);
            xr[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (gg < gcount) {
              if (e + 3 < mb) {
                const v4f_any v = __builtin_nontemporal_load(reinterpret_cast<const v4f_any*>(xp));
                xr[q] = make_float4(v.x, v.y, v.z, v.w);
              } else {
                if (e + 0 < mb) xr[q].x = xp[0];
                if (e + 1 < mb) xr[q].y = xp[1];
                if (e + 2 < mb) xr[q].z = xp[2];
              }
            }
          }
        }
      };
      load_x(0);
      // ---- phase 1 -------------------------------------------------------------------------
      // (Code'_s ends by position, Code_s by the bit position)
      const uint32_t lim = row + (kSparse ? kTileW : (ws < m ? min(kTileW, m - ws) : 0u));
      for (;;) {
        if (tw_pending && sfill - (~np >> 5) <= kStrRing - kPiece) {
          put_piece(tw);
          tw_pending = false;
        }
        if (!tw_pending && cur < kDone) {
          tw_pending = true;
          load_piece(sfill, tw);
        }
        const uint32_t np_lim = ~((sfill - 1u) * 32u);   // np above it: both words are in the ring
#pragma unroll 1
        for (uint32_t t = 0; t < kSteps; ++t) {
          const bool c1 = cur < lim, c2 = np > np_lim;
          if ((__builtin_amdgcn_ballot_w64(c1) & __builtin_amdgcn_ballot_w64(c2)) == 0) break;
          if (c1 & c2) {
            uint32_t w = peek();
            constexpr uint32_t kSel = (kTabSize - 1u) << 3;
            v2u e = *lds_at<v2u>(tab + (((w >> (29u - kTabBits)) & kSel) | st));
            put_entry(e);
#pragma unroll
            for (uint32_t l = 1; l < kLooks; ++l) {
              if (cur < lim) {
                w <<= e.y & kTabLen;
                e = *lds_at<v2u>(tab + (((w >> (29u - kTabBits)) & kSel) | st));
                put_entry(e);
              }
            }
            // an entry of length 0: the string's end, or one token through the general reader
            if ((e.y & kTabLen) == 0) {
              if (kSparse && np == np_end) {
                cur += kDoneFlag;
              } else if (np > np_lim) {
                const uint32_t v = peek();
                uint32_t l;
                if (kSparse && st == 0) {
                  const uint32_t gap = omega_peek3(v, l);
                  if (gap == 0) {
                    bad = 1; cur += kDoneFlag;
                  } else {
                    np -= l; cur += gap - 1u; st = kTabState;
                  }
                } else {
                  uint32_t lev = omega_peek3(v << 1, l);
                  const bool ok = lev != 0 && (kSparse ? lev <= s : lev <= s + 1u);
                  if (!ok) {
                    bad = 1; cur += kDoneFlag;
                  } else {
                    if (!kSparse) lev -= 1u;
                    const uint32_t byte = (v >> 31) ? 0u - lev : lev;
                    if (kSparse) {
                      *lds_at<uint8_t>(cur) = (uint8_t)byte;
                      cur += 1u; st = 0;
                    } else {
                      part |= (byte & 0xFFu) << ((cur << 3) & 24u);
                      *lds_at<uint32_t>(cur & ~3u) = part;
                      cur += 1u;
                      part = (cur & 3u) ? part : 0u;
                    }
                    np -= 1u + l;
                  }
                }
              }
            }
          }
        }
        if (__builtin_amdgcn_ballot_w64(cur < lim) == 0) break;
      }
      if (!kSparse) {   // the word the cursor stands in: the bucket may end in it
        if (cur - row < kRowBytes) *lds_at<uint32_t>(cur & ~3u) = part;
      }
      wave_fence();
      // ---- phase 2 -------------------------------------------------------------------------
      for (uint32_t g0 = 0; g0 < gcount; g0 += 2u * NP) {
        if (g0) load_x(g0);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const uint32_t gg = g0 + 2u * q + half;
          const uint32_t src = (gg * K) & 63u;
          const uint32_t base = (uint32_t)__shfl((int)base32, (int)src, kWave);
          const uint32_t mb = (uint32_t)__shfl((int)m, (int)src, kWave);
          if (gg < gcount) {
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            uint32_t p = tile + gg * K * kRowBytes + i4;
            uint32_t sp = scales + 4u * gg * K4;
            auto term = [&](uint32_t w, float sc) {
              sum.x += sc * (float)(int)(int8_t)w;         // sign * (scale * level), Eq. (2)
              sum.y += sc * (float)(int)(int8_t)(w >> 8);
              sum.z += sc * (float)(int)(int8_t)(w >> 16);
              sum.w += sc * (float)(int)(int8_t)(w >> 24);
            };
            auto word = [&](uint32_t j) { return *lds_at<uint32_t>(p + j * kRowBytes); };
            uint32_t kk = 0;
            if (records_only) {
              for (; kk < K; ++kk) {
                const uint32_t w = word(0);
                const float sc = *lds_at<float>(sp);
                if ((int8_t)w) sum.x += sc * (float)(int)(int8_t)w;
                if ((int8_t)(w >> 8)) sum.y += sc * (float)(int)(int8_t)(w >> 8);
                if ((int8_t)(w >> 16)) sum.z += sc * (float)(int)(int8_t)(w >> 16);
                if ((int8_t)(w >> 24)) sum.w += sc * (float)(int)(int8_t)(w >> 24);
                p += kRowBytes;
                sp += 4u;
              }
            }
            for (; kk + 4u <= K; kk += 4u) {
              const v4f s4 = *lds_at<v4f>(sp);
              const uint32_t w0 = word(0), w1 = word(1), w2 = word(2), w3 = word(3);
              p += 4u * kRowBytes;
              sp += 16u;
              term(w0, s4.x); term(w1, s4.y); term(w2, s4.z); term(w3, s4.w);
            }
            for (; kk < K; ++kk) {
              term(word(0), *lds_at<float>(sp));
              p += kRowBytes;
              sp += 4u;
            }
            const uint32_t e = ws + i4;
            float* xp = a.x + ((uint64_t)base + e);
            float4 v = xr[q];
            if (a.step) {
              v.x = fmaf(-a.c, sum.x, v.x); v.y = fmaf(-a.c, sum.y, v.y);
              v.z = fmaf(-a.c, sum.z, v.z); v.w = fmaf(-a.c, sum.w, v.w);
            } else {
              v.x += sum.x; v.y += sum.y; v.z += sum.z; v.w += sum.w;
            }
            if (whole || e + 3 < mb) {
              v4f_any o; o.x = v.x; o.y = v.y; o.z = v.z; o.w = v.w;
              __builtin_nontemporal_store(o, reinterpret_cast<v4f_any*>(xp));
            } else {
              if (e + 0 < mb) xp[0] = v.x;
              if (e + 1 < mb) xp[1] = v.y;
              if (e + 2 < mb) xp[2] = v.z;
            }
          }
        }
      }
      wave_fence();
      // ---- clear the tile; what was decided past the window opens the next one ----------------
      if (kSparse) {   // (Code'_s stores every word of every row)
        const uint32_t past = *lds_at<uint32_t>(row + kTileW);
        wave_fence();
        v4u z = {0, 0, 0, 0};
#pragma unroll
        for (uint32_t j = 0; j < kTileBytes / 1024u; ++j) *lds_at<v4u>(tile + 1024u * j + 16u * lane) = z;
        if (kTileBytes % 1024u && (uint32_t)lane < (kTileBytes % 1024u) / 16u)
          *lds_at<v4u>(tile + kTileBytes / 1024u * 1024u + 16u * lane) = z;
        wave_fence();
        if (ws + kTileW < a.d) *lds_at<uint32_t>(row) = past;
      } else if (ws + kTileW >= m && cur < kDone) {
        cur += kDoneFlag;
      }
      cur -= kTileW;
    }
    // a valid Code_s string has ended exactly, inside the bucket
    if (kSparse && open) {
      const uint32_t c = (cur + (a.d + kTileW - 1) / kTileW * kTileW - row) & (kDoneFlag - 1u);
      if (np != np_end || c > m || st != 0) bad = 1;
    }
    if (bad) flag_corrupt(a.status);
    wave_fence();
  }
}

namespace {

template <int CODE>
hipError_t launch_tile(const DecodeArgs& a, uint32_t blocks, uint32_t waves, hipStream_t st) {
  const dim3 grid(blocks), block(64 * waves);
  const size_t lds = waves * (size_t)kWaveBytes + kFlagBytes;
  if (a.gw <= 2) hipLaunchKernelGGL((k_decode_tile<CODE, 1>), grid, block, lds, st, a);
  else if (a.gw <= 4) hipLaunchKernelGGL((k_decode_tile<CODE, 2>), grid, block, lds, st, a);
  else hipLaunchKernelGGL((k_decode_tile<CODE, 4>), grid, block, lds, st, a);
  return hipGetLastError();
}

}  // namespace

uint32_t tile_max_waves(uint32_t code) {
  const uint32_t table = 8u * (code == QSGD_CODE_SPARSE ? tab_entries<QSGD_CODE_SPARSE>()
                                                        : tab_entries<QSGD_CODE_DENSE>());
  const uint32_t fit = (160u * 1024u - table - kFlagBytes) / kWaveBytes;
  return fit < kTileMaxWaves ? fit : kTileMaxWaves;
}

hipError_t launch_decode_tile(const DecodeArgs& a, uint32_t blocks, uint32_t waves,
                              hipStream_t st) {
  if (a.code == QSGD_CODE_SPARSE) return launch_tile<QSGD_CODE_SPARSE>(a, blocks, waves, st);
  return launch_tile<QSGD_CODE_DENSE>(a, blocks, waves, st);
}

}  // namespace qsgd
