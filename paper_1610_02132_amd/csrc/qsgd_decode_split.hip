// Elias codes, few strings: every word, or every bit, of a string has a lane.
//
// A prefix code can only be read from its start, so the other decoders give every string a
// lane; below some ten thousand strings most of the machine then waits for the longest chain of
// records.  Here a lane takes 32 bits.  It starts to read at their first bit, as if a record
// began there, and stops at the first record boundary behind them.  Then it compares where it
// started with where the lane below stopped, and reads again from there if the two differ, until
// no lane has to: the string's first lane starts at a true boundary, so by induction every lane
// does then.  Prefix codes fall into step by themselves within a few records (five to nine rounds
// for records of 8 bits, three to five for records of 4); a damaged string takes at most one
// round per lane.  A prefix sum of the positions passed gives every lane its place, and a last
// walk writes signed levels as bytes into the message's row in LDS.  The rows of a bucket are then
// added up in message order in registers, as in the tile decoder.
//
// Where the machine has lanes to spare (BITS), nobody walks to fall into step: a lane for every BIT
// reads the one record that would begin there, and three rounds of "where does the record at my
// end lead" (records double each time) give every word a table of 32 entries, at which bit of the
// next word one arrives from each of its own.  A round is then one look-up in that table, and the
// last walk reads records that are in LDS already.
//
// `lanes` consecutive words of a string (16, 32 or 64) are a unit, which a part of a wavefront
// brings into step by itself; the units of a string exchange their ends through LDS.  A workgroup
// works on as many units at a time as it has room for, a bucket's strings one behind the other.
//
// Buckets above kEntryMinD carry a list of entry points, at most one per segment of kSeg positions: a
// workgroup then takes a segment, reads the stretch between two entry points that it lies in
// from every message, and checks that the stretch ends where the next one starts, at the
// position the list names.  The sums go to an accumulator, which is applied to x only if all
// strings were sound.
//
// A step of a walk looks up the next kBits bits in a table in LDS that holds up to two records;
// longer records are read by arithmetic.  Levels must fit a signed byte (s <= 127).
//
// Bound by latency.  A walk's step is an LDS look-up and some 20 dependent instructions, 0.2 us, and
// a round of a lane per word about 5 steps.  20 thousand values, d = 512, s = 4, K = 2 (records of 8
// bits), us from the kernel's start: table and strings 2.4 (3.9 while its loads waited one for the
// other), eight rounds 11, last walk 2, sum 1: 20.7 at first, 17.6 with the table's loads together.
// A lane per bit: 9.9.  It does some 50 instructions per word more, so that it loses where the
// machine is full: 4M values, d = 8192, s = 40, K = 4 188 us instead of 105.
// Step over K messages, with the header check (a lane per string, a thread per bucket for bucket
// sizes no vector load fits; a lane per word; a lane per bit):
//   20 thousand values, d = 8192, s = 40, K = 2     294 -> 42 us
//   1M values, d = 2124, s = 23 (max scale), K = 2  273 -> 74 us
//   2.1M values, d = 523, s = 3, K = 8              670 -> 35 us
//   573 thousand values in one bucket, Code'_s, s = 127, K = 7   17.6 ms -> 65 us
//   4M values, d = 100 thousand, s = 2, K = 16      1230 -> 268 us
//   100 thousand values, d = 512, s = 3, K = 8      34 -> 25 -> 17 us
//   1M values, d = 2048, s = 6, K = 2               72 -> 30 -> 18 us
// Pieces of up to seven words a lane, a wavefront to a string, took 68, 118 and 54 us on the first three.
#include <algorithm>
#include <type_traits>

#include "qsgd_device.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

namespace {

constexpr uint32_t kBits = 10;
constexpr uint32_t kEntries = 1u << kBits;

// How many bits the LAST group of the code word at the top of the kBits bits has after its leading
// 1 (7 bits settle it); the value is 2^more + those bits, if a 0 follows them.
constexpr uint32_t last_group(uint32_t bits) {
  uint32_t at = 0, N = 1, more = 0;
  for (uint32_t groups = 0; groups < 3 && ((bits >> (kBits - 1 - at)) & 1u); ++groups) {
    more = N;
    if (groups == 2) break;
    const uint32_t v = (bits >> (kBits - 1 - at - N)) & ((1u << (N + 1)) - 1u);
    at += N + 1;
    N = v;
  }
  return more;
}
// Entry: bits of one / of two records (0, 4), positions passed (8, 12: 4 and 5 bits), their
// signed levels (17, 22: 5 bits each).  A single record stands twice; length 0: none fits.  And
// last_group of the first code word (28; behind the sign in Code'_s, of the level).
constexpr uint32_t record_entry(bool sparse, uint32_t bits) {
  uint32_t used = 0, adv = 0, e = 0;
  const uint32_t more = last_group(sparse ? bits : (bits << 1) & (kEntries - 1u));
  for (uint32_t r = 0; r < 2; ++r) {
    uint32_t left = kBits - used, u = used, gap = 1;
    if (sparse) {
      const Token t = omega_of(bits & ((1u << left) - 1u), left);
      if (t.len == 0) break;
      gap = t.value; u += t.len; left -= t.len;
    }
    if (left < 2) break;
    const uint32_t neg = (bits >> (left - 1)) & 1u;
    const Token t = omega_of(bits & ((1u << (left - 1)) - 1u), left - 1);
    if (t.len == 0) break;
    u += 1 + t.len;
    const uint32_t lev = sparse ? t.value : t.value - 1;
    const uint32_t byte = (neg ? 0u - lev : lev) & 31u;
    used = u; adv += gap;
    if (r == 0) e = used | used << 4 | adv << 8 | adv << 12 | byte << 17 | byte << 22;
    else e = (e & ~(0xFu << 4 | 0x1Fu << 12 | 0x1Fu << 22)) | used << 4 | adv << 12 | byte << 22;
  }
  return e | more << 28;
}

template <int CODE>
struct alignas(16) Records {
  uint32_t e[kEntries];
  constexpr Records() : e() {
    for (uint32_t i = 0; i < kEntries; ++i) e[i] = record_entry(CODE == QSGD_CODE_SPARSE, i);
  }
};
__device__ const Records<QSGD_CODE_SPARSE> g_records_sparse;
__device__ const Records<QSGD_CODE_DENSE> g_records_dense;

__device__ __forceinline__ int32_t field5(uint32_t e, uint32_t at) {   // signed
  return (int32_t)(e << (27u - at)) >> 27;
}

// LDS, in words: rows, then per message of a batch (scale, address of the string, words, first and
// end bit, position before, position behind, first unit), a total, whether a string has several
// units, per unit (end of the last lane, positions passed), what the next turn goes on from, and
// the status word.  Then, per word of a turn: the record that begins at each of its bits, where the
// records from each of its bits on leave it, and the word itself with the two behind it.
constexpr uint32_t kPerRow = 9, kPerUnit = 2, kMore = 5;
constexpr uint32_t kPerWord = 32 + 8 + 3;
constexpr uint32_t kLast = 0xFFFFFFFFu;   // position behind: the string's end, wherever it is

// The last of `ents` entry points (bit, position before it) at or before position P; 0: the
// string's start.  (A damaged list gives some number in range, the same one for everybody.)
__device__ __forceinline__ uint32_t entry_before(const uint32_t* list, uint32_t ents, uint32_t P) {
  uint32_t lo = 0, hi = ents;
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo + 1u) / 2u;
    if (list[2ull * mid - 1u] <= P) lo = mid; else hi = mid - 1u;
  }
  return lo;
}

}  // namespace

// A workgroup per bucket at a time; LONGB (buckets above kEntryMinD): per segment of kSeg positions.
template <int CODE, int NG, bool LONGB, bool BITS>
__global__ __launch_bounds__(64 * kSplitWaves) void k_decode_split(DecodeArgs a) {
  constexpr bool kSparse = CODE == QSGD_CODE_SPARSE;
  __shared__ __attribute__((aligned(16))) uint32_t table[kEntries];   // (filled 16 bytes at a time)
  const uint32_t status = *a.status;
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  const uint32_t thread = threadIdx.x, threads = blockDim.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(thread >> 6);
  // (the thread's number is made anew in every part: what can be worked out from it would else be
  // kept in registers from one end of the kernel to the other, and cost half of the wavefronts)
  auto afresh = [](uint32_t v) { asm volatile("" : "+v"(v)); return v; };
  const uint32_t K = a.K, s = a.s, rows = a.rows, lanes = a.lanes;
  const uint32_t row_words = LONGB ? kSeg / 4u : (a.d + 3u) / 4u;
  float* const scales = reinterpret_cast<float*>(smem + rows * row_words);
  uint32_t* const s_str = smem + rows * (row_words + 1u);   // low and high half of the address
  uint32_t* const s_words = s_str + 2u * rows;
  uint32_t* const s_begin = s_words + rows;
  uint32_t* const s_end = s_begin + rows;
  uint32_t* const s_prev = s_end + rows;
  uint32_t* const s_next = s_prev + rows;
  uint32_t* const s_unit = s_next + rows;            // rows + 1 of them
  // words worked on at a time, and units (`lanes` is 16, 32 or 64: a division by it in every turn took
  // 3% of a step of Code'_s)
  const uint32_t turn_words = BITS ? a.turn_words : threads;
  const uint32_t lane_bits = 31u - (uint32_t)__builtin_clz(lanes);
  const uint32_t slots = turn_words >> lane_bits;
  uint32_t* const s_several = s_unit + rows + 1u;
  uint32_t* const carry = s_several + 1;             // 2: entry and position of the next turn's first unit
  uint32_t* const u_exit = carry + 2;
  uint32_t* const u_adv = u_exit + slots;
  uint32_t* const damaged = u_adv + slots;
  uint32_t* const recs = damaged + 1;
  uint8_t* const leaves = reinterpret_cast<uint8_t*>(recs + 32u * turn_words);
  uint32_t* const w_words = recs + 40u * turn_words;
  const uint64_t pay = (uint64_t)H_WORDS + a.table_words;

  for (uint32_t i = thread; i < rows * row_words; i += threads) smem[i] = 0;
  bool opened = false;   // the table is in LDS

  const uint32_t segs = LONGB ? (a.d - 1u) / kSeg + 1u : 1u;   // (a.nb * segs < 2^32)
  for (uint32_t task = blockIdx.x; task < a.nb * segs; task += gridDim.x) {
    const uint32_t b = LONGB ? task / segs : task, P = LONGB ? (task - b * segs) * kSeg : 0u;
    uint64_t base;
    uint32_t M;
    bucket_extent(a, b, base, M);
    if (LONGB && P >= M) continue;
    const uint32_t m = LONGB ? min(kSeg, M - P) : M;   // positions P + 1 .. P + m of the bucket's M
    base += P;
    float* const x = (LONGB ? a.acc : a.x) + base;
    float4 xr[NG], sum[NG];
    const uint32_t first4 = 4u * afresh(thread);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t e = first4 + 4u * (uint32_t)i * threads;
      xr[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (LONGB) continue;
      if (e + 3 < m) {
        const v4f_any v = *reinterpret_cast<const v4f_any*>(x + e);
        xr[i] = make_float4(v.x, v.y, v.z, v.w);
      } else {
        if (e + 0 < m) xr[i].x = x[e];
        if (e + 1 < m) xr[i].y = x[e + 1];
        if (e + 2 < m) xr[i].z = x[e + 2];
      }
    }
    for (uint32_t k0 = 0; k0 < K; k0 += rows) {
      const uint32_t kn = min(rows, K - k0);
      // (the table's loads are under way while the first strings are opened)
      uint4 entries[kEntries / 256];
      const uint32_t tid = afresh(thread), lane = tid & 63u;
      if (!opened) {
        const uint4* src;
        if constexpr (kSparse) src = reinterpret_cast<const uint4*>(g_records_sparse.e);
        else src = reinterpret_cast<const uint4*>(g_records_dense.e);
#pragma unroll
        for (uint32_t j = 0; j < kEntries / 256; ++j) entries[j] = src[min(tid + j * threads, kEntries / 4u - 1u)];
      }
      // ---- open the strings ---------------------------------------------------------------
      if (wave == 0) {
        uint32_t units = 0;
        if (lane < kn) {
          const uint32_t* const msg = a.msgs[k0 + lane];
          const uint64_t msg_words = a.msg_words[k0 + lane];
          // (the header check may have found the message too short for its table, and its word
          // has not been looked at yet)
          const bool has_table = msg_words >= pay;
          const uint32_t o0 = has_table ? msg[H_WORDS + b] : 0u, o1 = has_table ? msg[H_WORDS + b + 1] : 0u;
          bool open = o0 < o1 && pay + o1 <= msg_words;
          uint32_t begin = 32, endbit = 0, first = 0, words = 0, prev = 0, next = kLast;
          const uint32_t* const str = msg + (pay + o0);
          if (open) {
            first = str[0];
            words = o1 - o0;
            uint32_t ents = 0;
            if (LONGB) {
              ents = str[words - 1u];
              open = 2ull * ents + 1u < words;
              words = open ? words - (2u * ents + 1u) : 1u;
            }
            endbit = words * 32u;
            if (kSparse) {
              const uint32_t last = str[words - 1u];
              endbit -= 1u + (uint32_t)(__ffs((int)last) - 1);
              open = open && last != 0 && endbit >= 32u;
            } else {
              open = open && endbit > 32u;
            }
            if (LONGB && open) {
              // the stretch between two entry points that this segment lies in; every stretch is
              // somebody's if the first segment's is the first, the next segment's the same or
              // the next, and the last segment's the last
              const uint32_t* const list = str + words;
              const uint32_t e = entry_before(list, ents, P);
              const uint32_t e2 = P + m < M ? entry_before(list, ents, P + kSeg) : ents;
              open = (P != 0 || e == 0) && (e2 == e || (e2 == e + 1u && P + m < M));
              if (e) { begin = list[2u * e - 2u]; prev = list[2u * e - 1u]; }
              uint32_t stop = endbit;
              if (e < ents) { stop = list[2u * e]; next = list[2u * e + 1u]; }
              open = open && begin >= 32u && begin <= stop && stop <= endbit && prev <= M && next != prev;
              endbit = stop;
              if (begin == endbit && (next != kLast || (!kSparse && prev < M))) open = false;
            }
          }
          if (!open) flag_corrupt(a.status);
          scales[lane] = open ? __uint_as_float(first) / (float)s : 0.f;
          s_str[lane] = (uint32_t)(uintptr_t)str;
          s_str[rows + lane] = (uint32_t)((uint64_t)(uintptr_t)str >> 32);
          s_words[lane] = words;
          s_begin[lane] = begin;
          s_end[lane] = open ? endbit : 0u;
          s_prev[lane] = prev;
          s_next[lane] = next;
          // words that hold records (the first word of a string is the scale)
          words = open && begin < endbit ? (endbit + 31u) / 32u - begin / 32u : 0u;
          units = (words + lanes - 1u) / lanes;
        }
        const uint32_t incl = wave_incl_scan_u32(units, (int)lane);
        if (lane < kn) s_unit[lane] = incl - units;
        const bool several = __builtin_amdgcn_ballot_w64(units > 1u) != 0;
        if (lane == 63u) { s_unit[kn] = incl; *s_several = several; }
      }
      if (!opened) {
        auto stored = [&](uint32_t e) {   // (a level above s is for the general reader to refuse)
          return (uint32_t)abs(field5(e, 17)) > s || (uint32_t)abs(field5(e, 22)) > s ? e & 0xF0000000u : e;
        };
#pragma unroll
        for (uint32_t j = 0; j < kEntries / 256; ++j) {
          const uint32_t i = tid + j * threads;
          const uint4 e = entries[j];
          if (i < kEntries / 4u)
            reinterpret_cast<uint4*>(table)[i] = make_uint4(stored(e.x), stored(e.y), stored(e.z), stored(e.w));
        }
        if (tid == 0) *damaged = status;
      }
      __syncthreads();
      // (other workgroups set the status word meanwhile: a workgroup's wavefronts leave together)
      if (!opened && *damaged) return;
      opened = true;
      const bool several = *s_several != 0;
      const uint32_t total = s_unit[kn];
      for (uint32_t turn = 0; turn < total; turn += slots) {
        const uint32_t tid = afresh(thread), lane = tid & 63u;
        const uint32_t slot = tid >> lane_bits, l = lane & (lanes - 1u);
        const uint32_t u = turn + slot;
        const bool here = !BITS || tid < turn_words;
        const bool live = here && u < total;
        // the string this unit belongs to: the last one that starts at or before it
        uint32_t r = 0;
        for (uint32_t step = 32; step; step >>= 1)
          if (r + step < kn && s_unit[r + step] <= u) r += step;
        const uint32_t ui = u - s_unit[r];                     // unit of the string
        const uint32_t begin = LONGB ? s_begin[r] : 32u;
        const uint32_t wi = begin / 32u + ui * lanes + l;      // word of the string
        const uint32_t endbit = live ? s_end[r] : 0u;
        const uint32_t end = min(32u, endbit > 32u * wi ? endbit - 32u * wi : 0u);
        const bool idle = end == 0;                            // the string ends before this word
        const bool final_word = !idle && endbit <= 32u * wi + 32u;
        uint32_t w0 = 0, w1 = 0, w2 = 0;
        if (!idle) {
          const uint32_t* const str =
              reinterpret_cast<const uint32_t*>((uintptr_t)((uint64_t)s_str[rows + r] << 32 | s_str[r]));
          const uint32_t nwords = s_words[r];
          w0 = str[wi];
          w1 = wi + 1u < nwords ? str[wi + 1u] : 0u;
          w2 = wi + 2u < nwords ? str[wi + 2u] : 0u;
        }
        uint8_t* const row = reinterpret_cast<uint8_t*>(smem + r * row_words);
        const uint32_t next = LONGB ? s_next[r] : kLast;
        uint32_t entry = LONGB && l == 0 && ui == 0 ? begin & 31u : 0u, exit = 0, adv = 0;
        const bool goes_on = ui != 0;                          // behind another unit of its string
        if (l == 0 && goes_on && slot == 0) entry = carry[0];  // (known from the turn before)
        bool fail = false;
        // (a lane for every word: from its entry to the first record boundary behind the word)
        auto walk = [&](auto write, uint32_t start) {
          constexpr bool W = decltype(write)::value;
          const uint32_t h0 = w0 >> 1, h1 = __builtin_amdgcn_alignbit(w0, w1, 1);
          const uint32_t h2 = __builtin_amdgcn_alignbit(w1, w2, 1), h3 = w2 << 31;
          uint32_t o = entry, p = start;
          fail = false;
          while (o < end) {
            const uint32_t v1 = __builtin_amdgcn_alignbit(h0, h1, ~o);   // the 32 bits from bit o on
            const uint32_t e = table[v1 >> (32u - kBits)];
            const uint32_t len1 = e & 15u;
            if (len1) {
              const bool two = o + len1 < end;
              const uint32_t p1 = p + ((e >> 8) & 15u), p2 = p + ((e >> 12) & 31u);
              if (W) {
                if (p1 - 1u - P < m) row[p1 - 1u - P] = (uint8_t)field5(e, 17);
                if (two && p2 - 1u - P < m) row[p2 - 1u - P] = (uint8_t)field5(e, 22);
              }
              o += two ? (e >> 4) & 15u : len1;
              p = two ? p2 : p1;
            } else {
              uint32_t gap = 1, gl = 0, ll, lev, open = 0, v = v1, more = e >> 28;
              if (kSparse) {
                gap = by_last_group(v1, more, gl, open);
                if (open) gap = LONGB ? omega_loop(((uint64_t)w0 << 32 | w1) << o | ((uint64_t)w2 << o >> 32), gl) : 0u;
              }
              const uint32_t q = o + gl;                       // (gap, sign and level end below bit 96)
              if (kSparse) {
                const uint32_t hi = q < 32u ? h0 : q < 64u ? h1 : h2, lo = q < 32u ? h1 : q < 64u ? h2 : h3;
                v = __builtin_amdgcn_alignbit(hi, lo, ~q);
                more = table[v << 1 >> (32u - kBits)] >> 28;
              }
              if (kSparse || LONGB) {
                lev = by_last_group(v << 1, more, ll, open);
              } else {
                // (group by group: 17 thousand values, d = 3376, s = 39, K = 5 47.4 us, by the last one 48.4; segments
                // the other way round: 5M values, s = 127, max, K = 3 340 and 327)
                lev = omega_peek3(v << 1, ll);
                open = lev == 0 ? 1u : 0u;
              }
              if (gap == 0 || open || lev > (kSparse ? s : s + 1u) || (LONGB && gap > M)) { fail = true; break; }
              if (!kSparse) lev -= 1u;
              p += gap;
              if (W && LONGB && kSparse && p > M) { fail = true; break; }
              if (W) { if (p - 1u - P < m) row[p - 1u - P] = (uint8_t)((v >> 31) ? 0u - lev : lev); }
              o = q + 1u + ll;
            }
          }
          exit = fail ? max(end, entry) : o;
          adv = p - start;
        };
        if (BITS) {
          if (!idle) {
            w_words[tid] = w0;
            w_words[turn_words + tid] = w1;
            w_words[2u * turn_words + tid] = w2;
          }
          if (here && l == 0) u_exit[slot] = idle ? 0u : (endbit + 31u) / 32u - wi;   // words from here on
          __syncthreads();
        }
        // ---- a lane for every bit: the record that would begin there ----------------------------
        if (BITS) for (uint32_t t0 = wave * 2u; t0 < turn_words; t0 += threads / 32u) {
          if ((t0 & (lanes - 1u)) >= __builtin_amdgcn_readfirstlane(u_exit[t0 >> lane_bits])) continue;
          const uint32_t t = t0 + (lane >> 5), o = lane & 31u;
          const uint32_t w0 = w_words[t], w1 = w_words[turn_words + t], w2 = w_words[2u * turn_words + t];
          // the 32 bits from bit o on are alignbit(h0, h1, ~o)
          const uint32_t h0 = w0 >> 1, h1 = __builtin_amdgcn_alignbit(w0, w1, 1);
          const uint32_t v1 = __builtin_amdgcn_alignbit(h0, h1, ~o);
          const uint32_t e = table[v1 >> (32u - kBits)];
          uint32_t len = e & 15u, gap = (e >> 8) & 15u, lev = (uint32_t)field5(e, 17), to = o + len;
          if (len) {
            to = to < 32u ? o + ((e >> 4) & 15u) : to;
          } else {
            const uint32_t h2 = __builtin_amdgcn_alignbit(w1, w2, 1), h3 = w2 << 31;
            uint32_t q = o, v = v1, more = e >> 28, ll, open;
            bool good = true;
            if (kSparse) {
              uint32_t gl;
              gap = by_last_group(v1, more, gl, open);
              if (open) {
                gap = LONGB ? omega_loop(((uint64_t)w0 << 32 | w1) << o | ((uint64_t)w2 << o >> 32), gl) : 0u;
                good = gap != 0;
              }
              if (LONGB) good = good && gap <= M;
              q = o + gl;                                      // (gap, sign and level end below bit 96)
              const uint32_t hi = q < 32u ? h0 : q < 64u ? h1 : h2, lo = q < 32u ? h1 : q < 64u ? h2 : h3;
              v = __builtin_amdgcn_alignbit(hi, lo, ~q);
              more = table[v << 1 >> (32u - kBits)] >> 28;
            }
            lev = by_last_group(v << 1, more, ll, open);
            good = good && !open && lev <= (kSparse ? s : s + 1u);
            if (!kSparse) lev -= 1u;
            lev = (v >> 31) ? 0u - lev : lev;
            len = good ? q - o + 1u + ll : 0u;
            to = good ? o + len : 32u;
            if (!kSparse) gap = 1;
            if (LONGB && gap > 0xFFFFu) gap = 0;               // (read again where it is used)
          }
          recs[t * 32u + o] = len ? len | (lev & 0xFFu) << 8 | gap << 16 : 0u;
          // Eight of these jumps leave the word from wherever they begin.  A jump of two records passes 6
          // bits at least.  One of a single record may pass 3, but then the record behind does not fit
          // in the rest of the kBits bits: these two jumps pass kBits + 1 = 11 at least.  (Where the
          // entry was dropped for a level above s, the record with that level ends the chain: `to` = 32.)
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const uint32_t on = (uint32_t)__shfl((int)to, (int)((lane & 32u) | (to & 31u)), kWave);
            to = to < 32u ? on : to;
          }
          leaves[t * 32u + o] = (uint8_t)to;
        }
        if (BITS) __syncthreads();
        // ---- a lane for every word: where its first record begins -------------------------------
        bool again = !idle;
        // (strings of one unit each need no look at the others' ends)
        for (uint32_t pass = 0; pass <= (several ? slots : 0u); ++pass) {
          for (uint32_t round = 0; round <= lanes; ++round) {
            if (again) {
              if constexpr (BITS) exit = entry < 32u ? leaves[tid * 32u + entry] : entry;
              else walk(std::false_type{}, 0u);
            }
            const uint32_t below = (uint32_t)__shfl_up((int)exit, 1, kWave) - 32u;
            const uint32_t now = l == 0 || idle ? entry : below;
            again = now != entry;
            entry = now;
            if (__builtin_amdgcn_ballot_w64(again) == 0) break;
          }
          if (!several) break;
          if (here && l == lanes - 1u) u_exit[slot] = exit - 32u;
          __syncthreads();
          if (l == 0 && live && goes_on && slot != 0) {
            const uint32_t now = u_exit[slot - 1u];
            again = now != entry;
            entry = now;
          }
          if (!__syncthreads_or(again)) break;
        }
        // ---- the word's records, and the positions they pass --------------------------------------
        constexpr int kMost = kSparse ? 11 : 16;
        uint32_t rec[kMost];
        // (a gap of 2^16 and more)
        auto far = [&](uint32_t at) {
          uint32_t n;
          return omega_loop(((uint64_t)w0 << 32 | w1) << at | ((uint64_t)w2 << at >> 32), n);
        };
        if constexpr (BITS) {
          const uint32_t leave = exit;
          exit = entry;
#pragma unroll
          for (int i = 0; i < kMost; ++i) {
            rec[i] = 0;
            if (exit < end && !fail) {
              rec[i] = recs[tid * 32u + exit];
              uint32_t gap = rec[i] >> 16;
              fail = rec[i] == 0;
              if (LONGB && kSparse && gap == 0 && !fail) gap = far(exit);
              adv += gap;
              exit += rec[i] & 0xFFu;
            }
          }
          exit = fail ? leave : exit;
        }
        uint32_t incl = adv;
        for (uint32_t t = 1; t < lanes; t <<= 1) {
          const uint32_t up = (uint32_t)__shfl_up((int)incl, t, kWave);
          if (l >= t) incl += up;
        }
        if (several) {
          if (here && l == lanes - 1u) u_adv[slot] = incl;
          __syncthreads();
        }
        uint32_t start = incl - adv;
        if (goes_on && live) {
          for (uint32_t t = slot; t > slot - min(ui, slot); --t) start += u_adv[t - 1u];
          if (ui > slot) start += carry[1];
        }
        if (LONGB && ui <= slot) start += s_prev[r];
        if (several) {
          __syncthreads();                     // carry is read, and may be written now
          if (slot == slots - 1u && l == lanes - 1u) { carry[0] = exit - 32u; carry[1] = start + adv; }
        }
        if (!idle) {
          const uint32_t exit_was = exit;
          if constexpr (BITS) {
            uint32_t p = start, at = entry;
            bool over = false;
#pragma unroll
            for (int i = 0; i < kMost; ++i) {
              if (rec[i]) {
                uint32_t gap = rec[i] >> 16;
                if (LONGB && kSparse && gap == 0) gap = far(at);
                at += rec[i] & 0xFFu;
                // (not the new position <= M: it is counted in 32 bits and could come round)
                over = over || (kSparse && gap > M - p);
                p += gap;
                if (!over && p - 1u - P < m) row[p - 1u - P] = (uint8_t)(rec[i] >> 8);
              }
            }
            fail = fail || over;
          } else {
            walk(std::true_type{}, start);
          }
          bool bad;
          // (every lane asks: positions are counted in 32 bits and could come round by the last one)
          if (kSparse || next != kLast)
            bad = fail || start + adv > M || (final_word && (exit_was != end || (next != kLast && start + adv != next)));
          // (what stands behind the bucket's last record of Code'_s is padding)
          else
            bad = (fail && start + adv < M) || (final_word && start + adv < M) ||
                  (final_word && exit_was > end && adv && start + adv <= M);
          if (bad) flag_corrupt(a.status);
        }
        if (turn + slots < total) __syncthreads();   // carry, before it is read
      }
      __syncthreads();
      // ---- add up the rows in message order, and clear them -------------------------------------
      // (zeros are left out where no term belongs: it matters to a scale that is not finite)
      const bool records_only = LONGB || kSparse || a.d % 4u != 0;
      const uint32_t g0 = afresh(thread);
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const uint32_t g = g0 + (uint32_t)i * threads;
        if (4u * g < m) {
          uint32_t* p = smem + g;
          for (uint32_t r = 0; r < kn; ++r, p += row_words) {
            const uint32_t w = *p;
            *p = 0;
            const float sc = scales[r];
            if (!records_only || w) {
              const int32_t l0 = (int8_t)w, l1 = (int8_t)(w >> 8), l2 = (int8_t)(w >> 16), l3 = (int8_t)(w >> 24);
              if (!records_only || l0) sum[i].x += sc * (float)l0;
              if (!records_only || l1) sum[i].y += sc * (float)l1;
              if (!records_only || l2) sum[i].z += sc * (float)l2;
              if (!records_only || l3) sum[i].w += sc * (float)l3;
            }
          }
        }
      }
      __syncthreads();
    }
    const uint32_t last4 = 4u * afresh(thread);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t e = last4 + 4u * (uint32_t)i * threads;
      float4 v = xr[i];
      if (LONGB) {
        v = sum[i];
      } else if (a.step) {
        v.x = fmaf(-a.c, sum[i].x, v.x); v.y = fmaf(-a.c, sum[i].y, v.y);
        v.z = fmaf(-a.c, sum[i].z, v.z); v.w = fmaf(-a.c, sum[i].w, v.w);
      } else {
        v.x += sum[i].x; v.y += sum[i].y; v.z += sum[i].z; v.w += sum[i].w;
      }
      if (e + 3 < m) {
        v4f_any o; o.x = v.x; o.y = v.y; o.z = v.z; o.w = v.w;
        *reinterpret_cast<v4f_any*>(x + e) = o;
      } else {
        if (e + 0 < m) x[e] = v.x;
        if (e + 1 < m) x[e + 1] = v.y;
        if (e + 2 < m) x[e + 2] = v.z;
      }
    }
  }
}

namespace {

template <int CODE, bool LONGB, bool BITS>
hipError_t launch_split(const DecodeArgs& a, const SplitPlan& p, hipStream_t st) {
  const dim3 grid(p.blocks), block(64 * p.waves);
  const uint32_t ng = ((LONGB ? kSeg : a.d) + 256u * p.waves - 1) / (256u * p.waves);
  if (ng <= 1) hipLaunchKernelGGL((k_decode_split<CODE, 1, LONGB, BITS>), grid, block, p.lds, st, a);
  else if (ng <= 2) hipLaunchKernelGGL((k_decode_split<CODE, 2, LONGB, BITS>), grid, block, p.lds, st, a);
  else if (ng <= 4) hipLaunchKernelGGL((k_decode_split<CODE, 4, LONGB, BITS>), grid, block, p.lds, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
template <bool LONGB>
hipError_t launch_split(const DecodeArgs& a, const SplitPlan& p, hipStream_t st) {
  if (a.code != QSGD_CODE_SPARSE) return launch_split<QSGD_CODE_DENSE, LONGB, false>(a, p, st);
  return p.bits ? launch_split<QSGD_CODE_SPARSE, LONGB, true>(a, p, st)
                : launch_split<QSGD_CODE_SPARSE, LONGB, false>(a, p, st);
}

}  // namespace

// How the strings are read, and about how long that takes.  us, step over K messages without its
// header check, measured on 20 thousand to 1.5M normal values (a lane per bit / per word / per string):
//   Code_s, 18 words, 4096 strings          21 / 26 / 28      234 strings     10 / 17 / 22
//   Code_s, 14 words, 4688 strings          20 / 27 / 27      320 strings     14 / 22 / 31
//   Code_s, 45 words, 2344 strings          23 / 25 / 45      80 strings      13 / 20 / 46
//   Code_s, 5 words, 6250 strings            - / 19 / 12      418 strings     10 / 13 / 11
//   Code'_s, 50 words, 4688 strings          - / 16 / 29      160 strings      - / 12 / 32
SplitPlan plan_decode_split(const DecodeArgs& a, uint32_t cus, uint32_t words, uint32_t expected) {
  SplitPlan p;
  const bool lng = a.d > kEntryMinD, sparse = a.code == QSGD_CODE_SPARSE;
  const uint32_t span = lng ? kSeg : a.d;
  // (a stretch between entry points has some kEntryBits at least)
  if (lng) words = std::max((uint32_t)((uint64_t)words * kSeg / a.d), kEntryBits / 32u + 8u);
  // (strings differ: one that needs a second unit holds the whole workgroup up)
  const uint32_t most = words + words / 5 + 2;
  p.lanes = most > 32 ? 64 : most > 16 ? 32 : 16;
  const uint32_t row = (span + 3) / 4 * 4;
  const uint32_t tasks = a.nb * ((a.d - 1) / span + 1), per_cu = (uint32_t)(((uint64_t)tasks + cus - 1) / cus);
  // rows of all messages at once if half of a compute unit's LDS holds them, else in batches
  p.rows = std::max(1u, std::min(a.K, 72u * 1024u / row));
  // a lane for every word of a batch, and at most 16 positions per thread in the sum
  const uint32_t units = p.rows * ((words + p.lanes - 1) / p.lanes);
  const uint32_t word_waves = (units * p.lanes + 63) / 64;
  auto lds_bytes = [&](bool bits) {
    return 4 * (p.rows * (row / 4 + kPerRow) + kPerUnit * (p.turn_words / p.lanes) + kMore +
                (bits ? kPerWord * p.turn_words : 0));
  };
  // A lane for every bit: where records are long (two bits per value at most: the words of
  // shorter ones fall into step as fast), and the buckets of a compute unit are all there at once
  // and not too much for its wavefronts: six per SIMD share the work.
  p.turn_words = 64 * word_waves;
  const uint64_t cu_words = (uint64_t)per_cu * a.K * words;
  p.bits = sparse && 16u * words <= span && p.rows == a.K && word_waves <= 12 && cu_words <= 700 &&
           (uint64_t)per_cu * (lds_bytes(true) + 4 * kEntries) <= 156u * 1024u;
  p.waves = p.bits ? std::max(word_waves, std::min(std::min(kSplitWaves, 24u / per_cu), (a.K * words + 1) / 2))
                   : std::min(kSplitWaves, word_waves);
  // Segments: the more of them, the smaller the workgroups, which wait for each other less; where a
  // compute unit has a single one, it gets all the wavefronts it can use.  479 steps over 20 thousand to 10M
  // values, both codes, K = 1 .. 16; time over that of the best of 16, 12, 8, 4 and 2 wavefronts, by
  // segments per compute unit:
  //            16     12     8      4                  16     12     8      4
  //   1        1.00   1.06   1.18   1.54     8 .. 15   1.18   1.09   1.08   1.01
  //   2, 3     1.11   1.01   1.05   1.28     16 ..     1.24   1.11   1.14   1.05
  //   4, 5     1.09   1.02   1.03   1.07
  //   6, 7     1.14   1.05   1.03   1.03
  // (16M values, d = 9770, Code'_s, s = 85, K = 4, 62 per compute unit: 16 / 8 / 4 / 2 693 / 625 / 593 / 491 us; 13M,
  // one bucket, s = 4, K = 8 349 / 349 / 321 / 368; many messages have the units for eight where there are eight
  // segments: 4M, d = 100 thousand, s = 2, K = 16 321 / 254 / 277 / 442.)
  if (lng && !p.bits)
    p.waves = std::min(p.waves, per_cu >= 16 ? std::max(2u, std::min(4u, a.K / 2)) : per_cu >= 8 ? (a.K >= 12 ? 8u : 4u)
                                : per_cu >= 6 ? 8u : per_cu >= 2 ? 12u : 16u);
  p.waves = std::max(p.waves, (span + 1023) / 1024);
  if (!p.bits) p.turn_words = 64 * p.waves;
  p.lds = lds_bytes(p.bits);
  const uint32_t fit = std::max(1u, std::min(32u / p.waves, 156u * 1024u / (p.lds + 4 * kEntries)));
  p.blocks = std::min(tasks, cus * fit);
  // (the whole step, header check and all; fitted like the other decoders' estimates, where the choice is made)
  if (p.bits) {
    p.us = 13.2 + 0.0372 * (double)per_cu * a.K * expected;
  } else {
    // the turns of a workgroup one after the other, and the words of a compute unit's buckets; a second
    // unit of a string costs both
    const uint32_t ups = (expected + p.lanes - 1) / p.lanes;   // units per string
    auto turns = [&](uint32_t n) { return (n * ups * p.lanes + 64 * p.waves - 1) / (64 * p.waves); };
    const double serial = (double)((tasks - 1) / p.blocks + 1) * (double)(a.K / p.rows * turns(p.rows) + turns(a.K % p.rows));
    const double work = (double)per_cu * a.K, values = (double)span;
    p.us = 11.9 + serial * (sparse ? 6.96 : 6.57) * (ups > 1 ? 1.21 : 1.0) +
           work * ((double)(ups * p.lanes) * (sparse ? 0.0061 : 0.0053) * (ups > 1 ? 1.93 : 1.0) + 3.8e-4 * values) +
           1.4e-6 * (double)tasks * values;
  }
  return p;
}

hipError_t launch_decode_split(DecodeArgs& a, const SplitPlan& p, hipStream_t st) {
  a.lanes = p.lanes; a.rows = p.rows; a.turn_words = p.turn_words;
  return a.d > kEntryMinD ? launch_split<true>(a, p, st) : launch_split<false>(a, p, st);
}

}  // namespace qsgd
