// Elias codes, few strings: every word of a string has a lane.
//
// A prefix code can only be read from its start, so the other decoders give every string a
// lane; below some ten thousand strings most of the machine then waits for the longest chain of
// records.  Here a lane takes 32 bits.  It starts to read at their first bit, as if a record
// began there, and stops at the first record boundary behind them.  Then it compares where it
// started with where the lane below stopped, and reads again from there if the two differ, until
// no lane has to: the string's first lane starts at a true boundary, so by induction every lane
// does then.  Prefix codes fall into step by themselves within a few records, so three to five
// rounds are the rule for strings of some 15 to 50 words and five to ten for 450 to 950; a
// damaged string takes at most one round per lane.  A prefix sum of the positions passed gives every lane its place, and a last walk writes signed levels as bytes
// into the message's row in LDS.  The rows of a bucket are then added up in message order in
// registers, as in the tile decoder.
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
// Bound by the latency of a walk's steps (about 7 steps a round, an LDS look-up and some 20
// dependent instructions each).  Step over K messages, before (a lane per string, a thread per
// bucket for bucket sizes no vector load fits) and with this decoder:
//   20 thousand values, d = 8192, s = 40, K = 2     294 -> 42 us
//   1M values, d = 2124, s = 23 (max scale), K = 2  273 -> 74 us
//   2.1M values, d = 523, s = 3, K = 8              670 -> 35 us
//   573 thousand values in one bucket, Code'_s, s = 127, K = 7   17.6 ms -> 65 us
//   4M values, d = 100 thousand, s = 2, K = 16      1230 -> 291 us
// Pieces of up to seven words a lane, a wavefront to a string, took 68, 118 and 54 us.
#include <algorithm>
#include <type_traits>

#include "qsgd_device.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

namespace {

constexpr uint32_t kBits = 10;
constexpr uint32_t kEntries = 1u << kBits;

// Entry: bits of one / of two records (0, 4), positions passed (8, 12: 4 and 5 bits), their
// signed levels (17, 22: 5 bits each).  A single record stands twice; length 0: none fits.
constexpr uint32_t record_entry(bool sparse, uint32_t bits) {
  uint32_t used = 0, adv = 0, e = 0;
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
  return e;
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

// LDS, in words: rows, then per message of a batch (scale, first word, words, first and end bit,
// position before, position behind, first unit), a total, per unit (end of the last lane,
// positions passed), what the next turn goes on from, and the status word.
constexpr uint32_t kPerRow = 8, kPerUnit = 2, kMore = 4;
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
template <int CODE, int NG, bool LONGB>
__global__ __launch_bounds__(64 * kSplitWaves) void k_decode_split(DecodeArgs a) {
  constexpr bool kSparse = CODE == QSGD_CODE_SPARSE;
  __shared__ uint32_t table[kEntries];
  const uint32_t status = *a.status;
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, threads = blockDim.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t K = a.K, s = a.s, rows = a.rows, lanes = a.lanes;
  const uint32_t row_words = LONGB ? kSeg / 4u : (a.d + 3u) / 4u;
  float* const scales = reinterpret_cast<float*>(smem + rows * row_words);
  uint32_t* const s_word = smem + rows * (row_words + 1u);
  uint32_t* const s_words = s_word + rows;
  uint32_t* const s_begin = s_words + rows;
  uint32_t* const s_end = s_begin + rows;
  uint32_t* const s_prev = s_end + rows;
  uint32_t* const s_next = s_prev + rows;
  uint32_t* const s_unit = s_next + rows;            // rows + 1 of them
  const uint32_t slots = threads / lanes;            // units worked on at a time
  uint32_t* const carry = s_unit + rows + 1u;        // 2: entry and position of the next turn's first unit
  uint32_t* const u_exit = carry + 2;
  uint32_t* const u_adv = u_exit + slots;
  uint32_t* const damaged = u_adv + slots;
  const uint32_t slot = tid / lanes, l = lane & (lanes - 1u);
  const uint64_t pay = (uint64_t)H_WORDS + a.table_words;

  {
    const uint32_t* src;
    if constexpr (kSparse) src = g_records_sparse.e; else src = g_records_dense.e;
    for (uint32_t i = tid; i < kEntries; i += threads) {
      uint32_t e = src[i];   // (a level above s is for the general reader to refuse)
      if ((uint32_t)abs(field5(e, 17)) > s || (uint32_t)abs(field5(e, 22)) > s) e = 0;
      table[i] = e;
    }
    for (uint32_t i = tid; i < rows * row_words; i += threads) smem[i] = 0;
    if (tid == 0) *damaged = status;
  }
  // (other workgroups set the status word meanwhile: a workgroup's wavefronts leave together)
  __syncthreads();
  if (*damaged) return;

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
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t e = 4u * (tid + (uint32_t)i * threads);
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
      // ---- open the strings ---------------------------------------------------------------
      if (wave == 0) {
        uint32_t units = 0;
        if (lane < kn) {
          const uint32_t* const msg = a.msgs[k0 + lane];
          const uint64_t msg_words = a.msg_words[k0 + lane];
          const uint32_t o0 = msg[H_WORDS + b], o1 = msg[H_WORDS + b + 1];
          bool open = o0 < o1 && pay + o1 <= msg_words;
          uint32_t begin = 32, endbit = 0, first = 0, words = 0, prev = 0, next = kLast;
          if (open) {
            const uint32_t* const str = msg + (pay + o0);
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
          s_word[lane] = o0;
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
        if (lane == 63u) s_unit[kn] = incl;
      }
      __syncthreads();
      const uint32_t total = s_unit[kn];
      for (uint32_t turn = 0; turn < total; turn += slots) {
        const uint32_t u = turn + slot;
        const bool live = u < total;
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
          const uint32_t* const str = a.msgs[k0 + r] + (pay + s_word[r]);
          const uint32_t nwords = s_words[r];
          w0 = str[wi];
          w1 = wi + 1u < nwords ? str[wi + 1u] : 0u;
          w2 = wi + 2u < nwords ? str[wi + 2u] : 0u;
        }
        uint8_t* const row = reinterpret_cast<uint8_t*>(smem + r * row_words);

        const uint32_t next = LONGB ? s_next[r] : kLast;
        uint32_t entry = LONGB && l == 0 && ui == 0 ? begin & 31u : 0u, exit = 0, adv = 0;
        bool fail = false;
        const bool goes_on = ui != 0;                          // behind another unit of its string
        if (l == 0 && goes_on && slot == 0) entry = carry[0];  // (known from the turn before)
        auto walk = [&](auto write, uint32_t start) {
          constexpr bool W = decltype(write)::value;
          uint32_t o = entry, p = start;
          fail = false;
          while (o < end) {
            const uint32_t v1 = (uint32_t)(((uint64_t)w0 << 32 | w1) << o >> 32);
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
              uint32_t gap = 1, ol = 0, ll;
              if (kSparse) gap = omega_peek3(v1, ol);
              if (LONGB && kSparse && gap == 0)                // (2^16 and more: up to 43 bits)
                gap = omega_loop(((uint64_t)w0 << 32 | w1) << o | ((uint64_t)w2 << o >> 32), ol);
              const uint32_t q = o + ol;                       // (gap, sign and level end below bit 96)
              const uint64_t pair = q < 32u ? ((uint64_t)w0 << 32 | w1)
                                  : q < 64u ? ((uint64_t)w1 << 32 | w2) : (uint64_t)w2 << 32;
              const uint32_t v = (uint32_t)(pair << (q & 31u) >> 32);
              uint32_t lev = omega_peek3(v << 1, ll);
              if (gap == 0 || lev == 0 || lev > (kSparse ? s : s + 1u) || (LONGB && gap > M)) { fail = true; break; }
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
        bool again = !idle;
        for (uint32_t pass = 0; pass <= slots; ++pass) {
          for (uint32_t round = 0; round <= lanes; ++round) {
            if (again) walk(std::false_type{}, 0u);
            const uint32_t below = (uint32_t)__shfl_up((int)exit, 1, kWave) - 32u;
            const uint32_t now = l == 0 || idle ? entry : below;
            again = now != entry;
            entry = now;
            if (__builtin_amdgcn_ballot_w64(again) == 0) break;
          }
          if (l == lanes - 1u) u_exit[slot] = exit - 32u;
          __syncthreads();
          if (l == 0 && live && goes_on && slot != 0) {
            const uint32_t now = u_exit[slot - 1u];
            again = now != entry;
            entry = now;
          }
          if (!__syncthreads_or(again)) break;
        }
        uint32_t incl = adv;
        for (uint32_t t = 1; t < lanes; t <<= 1) {
          const uint32_t up = (uint32_t)__shfl_up((int)incl, t, kWave);
          if (l >= t) incl += up;
        }
        if (l == lanes - 1u) u_adv[slot] = incl;
        __syncthreads();
        uint32_t start = incl - adv;
        if (goes_on) {
          for (uint32_t t = slot; t > slot - min(ui, slot); --t) start += u_adv[t - 1u];
          if (ui > slot) start += carry[1];
        }
        if (LONGB && ui <= slot) start += s_prev[r];
        const uint32_t exit_was = exit;
        __syncthreads();                       // carry is read, and may be written now
        if (slot == slots - 1u && l == lanes - 1u) { carry[0] = exit - 32u; carry[1] = start + adv; }
        if (!idle) {
          walk(std::true_type{}, start);
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
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const uint32_t g = tid + (uint32_t)i * threads;
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
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const uint32_t e = 4u * (tid + (uint32_t)i * threads);
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

template <int CODE, bool LONGB>
hipError_t launch_split(const DecodeArgs& a, uint32_t blocks, uint32_t waves, uint32_t lds, hipStream_t st) {
  const dim3 grid(blocks), block(64 * waves);
  const uint32_t ng = ((LONGB ? kSeg : a.d) + 256u * waves - 1) / (256u * waves);
  if (ng <= 1) hipLaunchKernelGGL((k_decode_split<CODE, 1, LONGB>), grid, block, lds, st, a);
  else if (ng <= 2) hipLaunchKernelGGL((k_decode_split<CODE, 2, LONGB>), grid, block, lds, st, a);
  else if (ng <= 4) hipLaunchKernelGGL((k_decode_split<CODE, 4, LONGB>), grid, block, lds, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_split(DecodeArgs& a, uint32_t cus, uint32_t words, hipStream_t st) {
  const bool lng = a.d > kEntryMinD;
  const uint32_t span = lng ? kSeg : a.d;
  // (a stretch between entry points has some kEntryBits at least)
  if (lng) words = std::max((uint32_t)((uint64_t)words * kSeg / a.d), kEntryBits / 32u + 8u);
  a.lanes = words > 32 ? 64 : words > 16 ? 32 : 16;
  const uint32_t row = (span + 3) / 4 * 4;
  // rows of all messages at once if half of a compute unit's LDS holds them, else in batches
  a.rows = std::max(1u, std::min(a.K, 72u * 1024u / row));
  // a lane for every word of a batch, and at most 16 positions per thread in the sum
  const uint32_t units = a.rows * ((words + a.lanes - 1) / a.lanes);
  uint32_t waves = std::min(kSplitWaves, (units * a.lanes + 63) / 64);
  waves = std::max(waves, (span + 1023) / 1024);
  const uint32_t lds = 4 * (a.rows * (row / 4 + kPerRow) + kPerUnit * (64 * waves / a.lanes) + kMore);
  const uint32_t fit = std::max(1u, std::min(32u / waves, 156u * 1024u / (lds + 4 * kEntries)));
  const uint32_t tasks = a.nb * ((a.d - 1) / span + 1);
  const uint32_t blocks = std::min(tasks, cus * fit);
  if (lng) return a.code == QSGD_CODE_SPARSE ? launch_split<QSGD_CODE_SPARSE, true>(a, blocks, waves, lds, st)
                                             : launch_split<QSGD_CODE_DENSE, true>(a, blocks, waves, lds, st);
  return a.code == QSGD_CODE_SPARSE ? launch_split<QSGD_CODE_SPARSE, false>(a, blocks, waves, lds, st)
                                    : launch_split<QSGD_CODE_DENSE, false>(a, blocks, waves, lds, st);
}

}  // namespace qsgd
