// Encode of Elias strings (d <= 8192): every lane codes its own values.
//
// Compacting the nonzero levels before they are coded costs more than it saves unless they are
// very rare.  Here a wavefront holds 64 / LPB buckets at once, LPB lanes each; a lane owns runs
// of 4 Q consecutive values, coalesced across the lanes.  Per run: Q Philox blocks, levels by
// Eq. (2), a prefix maximum over the bucket's lanes (where is the nonzero level before the
// lane's first one?), one look-up per value in a table in LDS that holds the whole code word
// of (gap, sign, level), the run's code words joined in a 64-bit register, a prefix sum of the
// lengths, and two or three ORs into the bucket's string in LDS.  The gap in front of a run's
// first nonzero level may be beyond the table and is then coded by arithmetic.  Levels from 32 on
// and runs of more than 64 bits look up gap and level one by one and go out four values at a
// time, two with levels from 64 on (where such levels are possible: LONG).  Above d = 2048 a
// bucket's runs do not fit the registers: they are read twice, the second time from the caches.
//
// Bound by instruction issue: on 25.6M values, s = 16, d = 512, 50 vector instructions per value
// and lane (of those Philox 10, rounding 8, code word 10) and 17 scalar ones, 0.8 vector
// instructions per SIMD and four clocks.  The same data 60 us through the survivor ring, 42
// directly; Code'_s 62 -> 36 us.
// A copy of the bytes would take 19 us.  Per encode, before and after: 57M values, d = 2124,
// s = 23 (max scale) 351 -> 187 us; 35M values, d = 4996, s = 11 153 -> 79 us.  (Kept in
// registers, 4 to 16 runs: 30M of d = 8192, s = 40 177 us instead of 89.)  Levels from 64 on, 10M
// values, largest value as scale, s = 255, d = 512 / 2048: Code_s 56 / 80 us through the survivor
// ring, 105 / 158 one value at a time from memory, 44 / 54 two at a time; Code'_s 48 / 54, 85 /
// 102, 35 / 43.  Bucket sizes that are no multiple of 4 pay a Philox
// block per run and two selects per draw word: 10M values, d = 443, s = 11, 33 us (47 with the words
// in scratch memory, 141 on the general path), d = 41 55 (71, 1150).
#include <type_traits>

#include "qsgd_device.hpp"
#include "qsgd_encode_wave.hpp"
#include "qsgd_kernels.hpp"

namespace qsgd {

namespace {

// Code word table: index gap * 64 + level * 2 + sign, entry (code << 8) | length; Code_s: gap 0
// stands for sign and level alone, level 0 has length 0 (also at the kGuard gaps below 0, which
// the zeros before a run's first nonzero level look up); Code'_s: gap 0 only.
constexpr uint32_t kGuard = 7, kMaxGap = 57, kMaxLev = 32;
// Elias code words of 1 .. kOmegas - 1, for longer runs of bits
constexpr uint32_t kOmegas = 128;

struct CodeLen { uint32_t code, len; };
constexpr CodeLen omega_word(uint32_t k) {
  uint32_t code = 0, len = 1;
  while (k > 1) {
    uint32_t nb = 0;
    for (uint32_t t = k; t; t >>= 1) ++nb;
    code |= k << len;
    len += nb;
    k = nb - 1;
  }
  return {code, len};
}

template <bool SPARSE> constexpr uint32_t code_entries() { return 2u * kMaxLev * (SPARSE ? kGuard + kMaxGap : 1u); }
template <bool SPARSE>
struct alignas(16) CodeTable {
  uint32_t e[code_entries<SPARSE>()], omega[kOmegas];
  constexpr CodeTable() : e(), omega() {
    for (uint32_t k = 1; k < kOmegas; ++k) omega[k] = omega_word(k).code << 8 | omega_word(k).len;
    for (uint32_t i = 0; i < code_entries<SPARSE>(); ++i) {
      const uint32_t row = i / (2 * kMaxLev), z = (i / 2) % kMaxLev, sign = i % 2;
      if (SPARSE && (z == 0 || row < kGuard)) { e[i] = 0; continue; }
      const uint32_t gap = SPARSE ? row - kGuard : 0;
      const CodeLen l = omega_word(SPARSE ? z : z + 1);
      uint32_t code = sign << l.len | l.code, len = l.len + 1;
      if (SPARSE && gap) {
        const CodeLen g = omega_word(gap);
        code |= g.code << len;
        len += g.len;
      }
      e[i] = code << 8 | len;
    }
  }
};
__device__ const CodeTable<true> g_codes_sparse;
__device__ const CodeTable<false> g_codes_dense;

// Inclusive scans over groups of LPB lanes (16, 32 or 64), and the value of the lane below
// (0 for the first lane of a group).
template <int LPB>
__device__ __forceinline__ uint32_t group_incl_sum(uint32_t v) {
  v += dpp_fetch<kDppShr1, 0xf>(v);
  v += dpp_fetch<kDppShr2, 0xf>(v);
  v += dpp_fetch<kDppShr4, 0xf>(v);
  v += dpp_fetch<kDppShr8, 0xf>(v);
  if (LPB >= 32) v += dpp_fetch<kDppBcast15, 0xa>(v);
  if (LPB >= 64) v += dpp_fetch<kDppBcast31, 0xc>(v);
  return v;
}
template <int LPB>
__device__ __forceinline__ uint32_t group_incl_max(uint32_t v) {
  v = max(v, dpp_fetch<kDppShr1, 0xf>(v));
  v = max(v, dpp_fetch<kDppShr2, 0xf>(v));
  v = max(v, dpp_fetch<kDppShr4, 0xf>(v));
  v = max(v, dpp_fetch<kDppShr8, 0xf>(v));
  if (LPB >= 32) v = max(v, dpp_fetch<kDppBcast15, 0xa>(v));
  if (LPB >= 64) v = max(v, dpp_fetch<kDppBcast31, 0xc>(v));
  return v;
}
template <int LPB>
__device__ __forceinline__ uint32_t group_lane_below(uint32_t v, uint32_t l) {
  const uint32_t up = dpp_fetch<kDppWaveShr1, 0xf>(v);
  return l == 0 ? 0u : up;
}
// Value of the group's last lane.
template <int LPB>
__device__ __forceinline__ uint32_t group_last(uint32_t v, int last_lane) {
  if (LPB == 64) return lane_bcast(v, 63);
  return (uint32_t)__shfl((int)v, last_lane, kWave);
}

}  // namespace

// ODD: bucket sizes that are no multiple of 4, whose buckets start anywhere in a Philox block.
// LONG: with the coder of long code words, which costs 25.6M values, s = 16, d = 512 50.1 -> 51.0
// us and d = 2048 55.6 -> 62.6; without it the few runs of more than 64 bits are read again by a
// small general coder.
// (Above d = 2048 the loads of the first reading would cost the fifth wavefront per SIMD: 20M values,
// s = 16, without / with the bound: d = 2052 60 / 55 us, 3000 53 / 54, 8192 72 / 73, Code'_s 53 / 49
// and 48 / 47.)
template <int LPB, int CP, int Q, int CODE, bool ODD, bool LONG>
__global__ __launch_bounds__(64 * kDirectWaves) __attribute__((amdgpu_waves_per_eu(CP == 0 ? 5 : 1)))
void k_encode_direct(EncodeArgs a) {
  constexpr bool kSparse = CODE == QSGD_CODE_SPARSE;
  constexpr uint32_t NB = 64 / LPB;             // buckets per wavefront pass
  constexpr int R = 4 * Q;                      // values of a run
  constexpr uint32_t kStep = LPB * R;           // values one run of the bucket's lanes covers
  constexpr uint32_t kTab = code_entries<kSparse>();
  __shared__ __attribute__((aligned(16))) uint32_t codes[kTab];
  __shared__ uint32_t omegas[LONG ? kOmegas : 1];
  extern __shared__ uint32_t smem[];            // per wavefront: NB bucket strings of dst_words
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const uint32_t sb = (uint32_t)lane / LPB, l = (uint32_t)lane % LPB;
  const int last_lane = (int)(sb * LPB + LPB - 1);
  uint32_t* const dst = smem + (wave * NB + sb) * a.dst_words;

  {
    const uint32_t *src, *om;
    if constexpr (kSparse) { src = g_codes_sparse.e; om = g_codes_sparse.omega; }
    else { src = g_codes_dense.e; om = g_codes_dense.omega; }
    // (16 bytes a load, all of them in flight)
    constexpr uint32_t kQuads = kTab / 4, kLoads = (kQuads + 64 * kDirectWaves - 1) / (64 * kDirectWaves);
    uint4 t[kLoads];
#pragma unroll
    for (uint32_t j = 0; j < kLoads; ++j)
      t[j] = reinterpret_cast<const uint4*>(src)[min((uint32_t)tid + j * 64u * kDirectWaves, kQuads - 1u)];
    if (LONG && tid < (int)kOmegas) omegas[tid] = om[tid];
    for (uint32_t j = l; j < a.dst_words; j += LPB) dst[j] = 0;
#pragma unroll
    for (uint32_t j = 0; j < kLoads; ++j) {
      const uint32_t i = (uint32_t)tid + j * 64u * kDirectWaves;
      if (i < kQuads) reinterpret_cast<uint4*>(codes)[i] = t[j];
    }
  }
  if (blockIdx.x == 0 && tid == 0) {  // header; length and status are completed later
    uint32_t* h = a.header;
    h[H_MAGIC] = kMagic; h[H_VERSION] = a.version; h[H_CODE] = CODE; h[H_NORM] = a.norm_mode;
    h[H_S] = a.s; h[H_STREAM] = a.stream_id;
    h[H_D_LO] = (uint32_t)a.d; h[H_D_HI] = 0;
    h[H_N_LO] = (uint32_t)a.n; h[H_N_HI] = (uint32_t)(a.n >> 32);
    h[H_NB_LO] = a.nb; h[H_NB_HI] = 0;
    h[H_PW_LO] = 0; h[H_PW_HI] = 0;
    h[H_STATUS] = 0; h[H_ITER] = a.iteration;
  }
  __syncthreads();

  const uint32_t team = blockIdx.x * kDirectWaves + wave;
  const uint32_t b_begin = team * a.bper;
  if (b_begin >= a.nb) return;
  const uint32_t b_end = min(b_begin + a.bper, a.nb);
  uint32_t* const region = a.staging + (uint64_t)team * a.region_words;
  uint32_t run = 0;  // words this team has appended to its region
  const uint32_t s = a.s;
  const float s_f = (float)s;
  const uint32_t zlim = min(s, kMaxLev - 1u);
  const uint32_t zlong = min(s, kSparse ? 63u : kOmegas - 2u);   // four values then fit 64 bits
  QuantCtx qc;
  qc.inv = 0.f; qc.s_f = s_f; qc.s = s; qc.key0 = a.key0; qc.key1 = a.key1;
  qc.stream_id = a.stream_id; qc.iteration = a.iteration;

  for (uint32_t b0 = b_begin; b0 < b_end; b0 += NB) {
    const uint32_t b = b0 + sb;
    const bool live = b < b_end;
    uint64_t base = 0;
    uint32_t m = 0;
    if (live) bucket_extent(a, b, base, m);
    const float* __restrict__ gb = a.g + base;
    const bool all_full = CP > 0 && __ballot(m == (uint32_t)CP * kStep) == ~0ull;
    // (CP = 0: one bucket at a time, its runs are read twice instead of kept in registers)
    const uint32_t runs = CP > 0 ? (uint32_t)CP : __builtin_amdgcn_readfirstlane((m + kStep - 1u) / kStep);

    auto load_four = [&](uint32_t e0, bool full) -> float4 {
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (full || e0 + 3 < m) {
        if constexpr (ODD) {
          const v4f_any t = *reinterpret_cast<const v4f_any*>(gb + e0);
          x = make_float4(t.x, t.y, t.z, t.w);
        } else {
          x = *reinterpret_cast<const float4*>(gb + e0);
        }
      } else {
        if (e0 + 0 < m) x.x = gb[e0 + 0];
        if (e0 + 1 < m) x.y = gb[e0 + 1];
        if (e0 + 2 < m) x.z = gb[e0 + 2];
      }
      return x;
    };
    auto load_run = [&](uint32_t at, bool full, float (&x8)[R]) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float4 x = load_four(at + l * R + 4 * q, full);
        x8[4 * q] = x.x; x8[4 * q + 1] = x.y; x8[4 * q + 2] = x.z; x8[4 * q + 3] = x.w;
      }
    };
    auto run_full = [&](uint32_t c) { return CP > 0 ? all_full : (c + 1u) * kStep <= m; };
    float v[CP > 0 ? CP : 1][R];
#pragma unroll
    for (int c = 0; c < CP; ++c) load_run((uint32_t)c * kStep, all_full, v[c]);

    // values [at, at + kShare) of a bucket above d = 2048, four at a time
    constexpr uint32_t kShare = 8 * kChunk;
    auto read_share = [&](uint32_t at, auto&& take) {
      if (at + kShare <= m) {   // (all of it requested together)
        float4 x[8];
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c) x[c] = load_four(at + c * kChunk + 4u * l, true);
#pragma unroll
        for (uint32_t c = 0; c < 8; ++c) take(x[c]);
      } else {
#pragma unroll 4
        for (uint32_t e = at; e < m; e += kChunk) take(load_four(e + 4u * l, false));
      }
    };

    // ---- scale of each bucket: reduction over its LPB lanes ------------------------------
    float scale;
    // (a bucket's sum of squares is taken in one order, whichever shape the number of buckets
    // picks: a slice has to get the whole vector's scales)
    if (a.norm_mode == 0) {
      double ss;
      auto square = [](float x, double sum) { return fma((double)x, (double)x, sum); };   // (exact in fp64)
      auto group_sum = [](double v) {   // right in the last lane of each bucket
        v += dpp_fetch_f64<kDppShr1, 0xf>(v);
        v += dpp_fetch_f64<kDppShr2, 0xf>(v);
        v += dpp_fetch_f64<kDppShr4, 0xf>(v);
        v += dpp_fetch_f64<kDppShr8, 0xf>(v);
        if (LPB >= 32) v += dpp_fetch_f64<kDppBcast15, 0xa>(v);
        if (LPB >= 64) v += dpp_fetch_f64<kDppBcast31, 0xc>(v);
        return v;
      };
      if constexpr (CP == 1) {
        // 64 < d <= 256: runs of four or eight.  Four values at a time, then pairwise by position:
        // a run of eight is what the first step of the lanes' tree adds up of two runs of four.
        double quad[Q];
#pragma unroll
        for (int t = 0; t < Q; ++t)
          quad[t] = square(v[0][4 * t + 1], square(v[0][4 * t], 0.0)) +
                    square(v[0][4 * t + 3], square(v[0][4 * t + 2], 0.0));
        ss = Q == 1 ? quad[0] : quad[0] + quad[Q - 1];
        ss = group_sum(ss);
      } else if constexpr (CP > 1) {   // (one shape per bucket size)
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
        for (int c = 0; c < CP; ++c) {
#pragma unroll
          for (int j = 0; j < R; j += 4) {
            s0 = square(v[c][j], s0);
            s1 = square(v[c][j + 1], s1);
            s2 = square(v[c][j + 2], s2);
            s3 = square(v[c][j + 3], s3);
          }
        }
        ss = group_sum((s0 + s1) + (s2 + s3));
      } else {
        // d > 2048: in the order of the encoder with a team of wavefronts per bucket, 2048 values
        // a wavefront, in chunks of 256
        ss = 0.0;
#pragma unroll 1
        for (uint32_t at = 0; at < m; at += kShare) {
          double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
          read_share(at, [&](const float4& x) {
            s0 = square(x.x, s0);
            s1 = square(x.y, s1);
            s2 = square(x.z, s2);
            s3 = square(x.w, s3);
          });
          ss += group_sum((s0 + s1) + (s2 + s3));
        }
      }
      scale = (float)sqrt(ss);  // right in the last lane of each bucket
    } else {
      float mx = 0.f;
      auto max_run = [&](const float (&x8)[R]) {
#pragma unroll
        for (int j = 0; j < R; ++j) mx = fmaxf(mx, fabsf(x8[j]));
      };
      if constexpr (CP > 0) {
#pragma unroll
        for (int c = 0; c < CP; ++c) max_run(v[c]);
      } else {
#pragma unroll 1
        for (uint32_t at = 0; at < m; at += kShare)
          read_share(at, [&](const float4& x) {
            mx = fmaxf(fmaxf(mx, fmaxf(fabsf(x.x), fabsf(x.y))), fmaxf(fabsf(x.z), fabsf(x.w)));
          });
      }
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr1, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr2, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr4, 0xf>(__float_as_uint(mx))));
      mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppShr8, 0xf>(__float_as_uint(mx))));
      if (LPB >= 32) mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppBcast15, 0xa>(__float_as_uint(mx))));
      if (LPB >= 64) mx = fmaxf(mx, __uint_as_float(dpp_fetch<kDppBcast31, 0xc>(__float_as_uint(mx))));
      scale = mx;
    }
    scale = __uint_as_float(group_last<LPB>(__float_as_uint(scale), last_lane));
    const float inv = (scale > 0.f) ? s_f / scale : 0.f;

    // ---- runs ---------------------------------------------------------------------------
    const uint64_t g0 = a.index_base + base + l * R;
    uint32_t hi;
    const bool uhi = uniform_counter_hi(g0, g0 + (uint64_t)(runs ? runs - 1u : 0u) * kStep + R - (ODD ? 0 : 4), hi);
    uint32_t bits = 32;        // bits of the bucket's string so far (the same in all its lanes)
    uint32_t last_pos = 0;     // 1-based position of the last nonzero level so far
    auto code_run = [&](const uint32_t c, const float (&x8)[R], const bool full) {
      // (one run after the other: side by side they cost the fifth wavefront per SIMD)
      __builtin_amdgcn_sched_barrier(0);
      uint32_t z[R], zmax = 0;
      uint32_t r[4 * (Q + ODD)];
#pragma unroll
      for (int q = 0; q < Q + ODD; ++q) {
        uint32_t r4[4];
        const uint64_t gi = g0 + (uint64_t)(c * kStep) + 4 * q;
        if (uhi) draw4_uniform_hi(gi, hi, qc, r4);
        else draw4<true>(gi, qc, r4);
#pragma unroll
        for (int j = 0; j < 4; ++j) r[4 * q + j] = r4[j];
      }
      if constexpr (ODD) {   // the run's first value has word g0 % 4 of the first block
        const bool one = (g0 & 1u) != 0, two = (g0 & 2u) != 0;
        // (values to choose from, not places: a choice of places keeps r in scratch memory)
        auto choose = [](bool take, uint32_t then, uint32_t other) { return take ? then : other; };
#pragma unroll
        for (int j = 0; j < R + 2; ++j) r[j] = choose(one, r[j + 1], r[j]);
#pragma unroll
        for (int j = 0; j < R; ++j) r[j] = choose(two, r[j + 2], r[j]);
      }
#pragma unroll
      for (int j = 0; j < R; ++j) {
        z[j] = quantize_unclamped(x8[j], inv, r[j]);
        zmax = max(zmax, z[j]);
      }
      const uint32_t e0 = c * kStep + l * R;     // bucket position of the run, 0-based
      // where the nonzero level before the run is; inside a run gaps are at most R, so only its
      // first one can be beyond the table
      uint64_t acc = 0;
      uint32_t len = 0, prev0 = 0, from = 0;
      if constexpr (kSparse) {
        uint32_t lastnz = 0;
#pragma unroll
        for (int j = 0; j < R; ++j) lastnz = z[j] ? (uint32_t)j + 1u : lastnz;
        const uint32_t im = group_incl_max<LPB>(lastnz ? e0 + lastnz : 0u);
        prev0 = max(group_lane_below<LPB>(im, l), last_pos);
        last_pos = max(last_pos, group_last<LPB>(im, last_lane));
        // (a run without a nonzero level looks up level 0 at gaps of the table all the same)
        from = lastnz ? prev0 : e0;
        const bool far = e0 + (uint32_t)R - from >= kMaxGap;
        if (__builtin_amdgcn_ballot_w64(far)) {
          // the gap's code word opens the run, its first level is looked up alone
          uint32_t firstnz = 0;
#pragma unroll
          for (int j = R - 1; j >= 0; --j) firstnz = z[j] ? (uint32_t)j + 1u : firstnz;
          if (far) {
            omega_encode(e0 + firstnz - prev0, acc, len);
            from = e0 + firstnz;
          }
        }
      }
      bool easy = __builtin_amdgcn_ballot_w64(zmax > zlim) == 0;
      if (easy) {
        // positions from the run's start on, in bytes of the table (2 kMaxLev words per gap); as
        // constants: positions in the bucket would be kept in 2 R registers over all buckets
        constexpr uint32_t kGapBytes = 8u * kMaxLev;
        uint32_t prev = (from - e0 - kGuard) * kGapBytes;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          uint32_t e;
          if constexpr (kSparse) {
            const uint32_t pos = ((uint32_t)j + 1u) * kGapBytes;
            const uint32_t zs = __builtin_amdgcn_alignbit(z[j], __float_as_uint(x8[j]), 31);   // z * 2 + sign
            e = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(codes) +
                                                   ((zs << 2) | (pos - prev)));
            prev = z[j] ? pos - kGuard * kGapBytes : prev;
          } else {
            const uint32_t zs = z[j] * 2u + (x8[j] < 0.f ? 1u : 0u);   // (-0.0 counts as positive)
            e = codes[zs];
            if (!full) e = e0 + (uint32_t)j < m ? e : 0u;
          }
          acc = (acc << (e & 63u)) | (e >> 8);
          len += e & 0xFFu;
        }
        easy = __builtin_amdgcn_ballot_w64(len > 64u) == 0;
      }
      if (easy) {
        const uint32_t incl = group_incl_sum<LPB>(len);
        if (len) lds_emit(dst, bits + incl - len, acc, len);
        bits += group_last<LPB>(incl, last_lane);
      } else if (LONG) {
        // long code words: gap and level looked up one by one, the first gap and every V values go
        // out by themselves: four values with levels up to zlong (at most 61 bits), else two (a
        // level of 2^16 in Code'_s has 28 bits, so at most 58)
        auto code_words = [&](auto values) {
          constexpr int V = decltype(values)::value, kParts = R / V;
          uint64_t gc = 0, part[kParts];
          uint32_t gl = 0, plen[kParts], first = 0, tot = 0, prev = 0;
          if constexpr (kSparse) {
#pragma unroll
            for (int j = R - 1; j >= 0; --j) first = z[j] ? (uint32_t)j + 1u : first;
            if (first) omega_encode(e0 + first - prev0, gc, gl);
            tot = gl;
          }
#pragma unroll
          for (int q = 0; q < kParts; ++q) {
            part[q] = 0; plen[q] = 0;
#pragma unroll
            for (int j = V * q; j < V * q + V; ++j) {
              if (kSparse ? z[j] != 0 : full || e0 + (uint32_t)j < m) {
                uint32_t k = (V == 4 ? z[j] : min(z[j], s)) + (kSparse ? 0u : 1u);
                uint32_t lw = omegas[V == 4 || k < kOmegas ? k : 31u - (uint32_t)__clz((int)k)];
                uint32_t code = lw >> 8, ll = lw & 0xFFu;
                if (V != 4 && k >= kOmegas) {   // the code word of its length, open, then k itself
                  const uint32_t nb = 32u - (uint32_t)__clz((int)k);
                  code = code >> 1 << (nb + 1u) | k << 1;
                  ll += nb;
                }
                if (kSparse && prev) {
                  const uint32_t gw = omegas[(uint32_t)j + 1u - prev];
                  part[q] = part[q] << (gw & 63u) | gw >> 8;
                  plen[q] += gw & 0xFFu;
                }
                part[q] = part[q] << (ll + 1u) | ((x8[j] < 0.f ? 1u : 0u) << ll | code);
                plen[q] += ll + 1u;
                prev = (uint32_t)j + 1u;
              }
            }
            tot += plen[q];
          }
          const uint32_t incl = group_incl_sum<LPB>(tot);
          uint32_t at = bits + incl - tot;
          if (gl) lds_emit(dst, at, gc, gl);
          at += gl;
#pragma unroll
          for (int q = 0; q < kParts; ++q) {
            if (plen[q]) lds_emit(dst, at, part[q], plen[q]);
            at += plen[q];
          }
          bits += group_last<LPB>(incl, last_lane);
        };
        if (__builtin_amdgcn_ballot_w64(zmax > zlong) == 0) code_words(std::integral_constant<int, 4>());
        else code_words(std::integral_constant<int, 2>());
      } else {
        // the general coder, from memory (rare with s < 32: kept small rather than fast, so that it
        // costs the usual path no registers): lengths, prefix sum, then one code word at a time
        uint32_t off = 0, incl = 0;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
          uint32_t prev = prev0, tot = 0;
#pragma unroll 1
          for (uint32_t j = 0; j < (uint32_t)R; ++j) {
            const uint32_t pos = e0 + j + 1u;
            if (pos > m) break;
            uint32_t r[4];
            const uint64_t gi = g0 + (uint64_t)(c * kStep) + j;
            draw4<true>(gi, qc, r);
            const uint32_t q = (uint32_t)gi & 3u;
            const float x = gb[pos - 1u];
            const uint32_t lev = quantize_one(x, inv, s_f, s, q == 0 ? r[0] : q == 1 ? r[1] : q == 2 ? r[2] : r[3]);
            if (kSparse && lev == 0) continue;
            uint64_t gc = 0, lc;
            uint32_t gl = 0, ll;
            if (kSparse) omega_encode(pos - prev, gc, gl);
            omega_encode(kSparse ? lev : lev + 1u, lc, ll);
            if (pass) {
              if (gl) lds_emit(dst, off + tot, gc, gl);
              lds_emit(dst, off + tot + gl, ((uint64_t)(x < 0.f ? 1u : 0u) << ll) | lc, ll + 1u);
            }
            tot += gl + ll + 1u;
            prev = pos;
          }
          if (pass == 0) {
            incl = group_incl_sum<LPB>(tot);
            off = bits + incl - tot;
          }
        }
        bits += group_last<LPB>(incl, last_lane);
      }
    };
    if constexpr (CP > 0) {
#pragma unroll
      for (int c = 0; c < CP; ++c) code_run((uint32_t)c, v[c], all_full);
    } else {
      float next[R];
      if (runs) load_run(0, run_full(0), next);
#pragma unroll 1
      for (uint32_t c = 0; c < runs; ++c) {
        float x8[R];
#pragma unroll
        for (int j = 0; j < R; ++j) x8[j] = next[j];
        if (c + 1u < runs) load_run((c + 1u) * kStep, run_full(c + 1u), next);
        code_run(c, x8, run_full(c));
      }
    }

    // ---- close the strings and append them to the team's region ----------------------------
    const uint32_t stop = kSparse ? 1u : 0u;
    const uint32_t words = live ? (bits + stop + 31u) >> 5 : 0u;
    if (l == 0 && live) {
      dst[0] = __float_as_uint(scale);
      if (kSparse) lds_emit(dst, bits, 1ull, 1u);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint32_t before = 0, all = words;
    if (NB > 1) {
      before = 0; all = 0;
#pragma unroll
      for (uint32_t t = 0; t < NB; ++t) {
        const uint32_t wt = lane_bcast(words, (int)(t * LPB));
        if (t < sb) before += wt;
        all += wt;
      }
    }
    // (a region smaller than the worst case may run out: the string is then dropped, the
    // count goes on, and the message ends up with the capacity status and the size needed)
    const uint32_t at = run + before;
    const bool room = (uint64_t)at + words <= a.region_words;
    if (l == 0 && live) a.table[b] = at;  // relative to the region; rebased later
    for (uint32_t j = l; j < words; j += LPB) {
      if (room) region[at + j] = dst[j];
      dst[j] = 0;
    }
    run += all;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0) a.totals[team] = run;
}

namespace {

template <int LPB, int CP, int Q, bool ODD, bool LONG>
hipError_t launch_code(const EncodeArgs& a, uint32_t code, uint32_t teams, hipStream_t st) {
  const dim3 grid((teams + kDirectWaves - 1) / kDirectWaves), block(64 * kDirectWaves);
  const size_t lds = 4 * (size_t)kDirectWaves * (64 / LPB) * a.dst_words;
  if (code == QSGD_CODE_SPARSE)
    hipLaunchKernelGGL((k_encode_direct<LPB, CP, Q, QSGD_CODE_SPARSE, ODD, LONG>), grid, block, lds, st, a);
  else
    hipLaunchKernelGGL((k_encode_direct<LPB, CP, Q, QSGD_CODE_DENSE, ODD, LONG>), grid, block, lds, st, a);
  return hipGetLastError();
}

// Levels that the table of code words does not hold, which a single large value brings about
// whatever the others are, or a mean level of normal values above one: with one or two bits of gap
// and sign, eight values are then close to 64 bits.
bool long_words(const EncodeArgs& a) {
  if (a.s >= kMaxLev) return true;
  const float scale = a.norm_mode ? sqrtf(2.f * logf((float)a.d + 2.f)) : sqrtf((float)a.d);
  return 0.8f * (float)a.s > 1.2f * scale;
}

template <int LPB, int CP, int Q, bool ODD = false>
hipError_t launch_direct(const EncodeArgs& a, uint32_t code, uint32_t teams, hipStream_t st) {
  // (runs read twice have the registers, and bucket sizes off the usual ones don't need two kernels)
  if constexpr (ODD || CP == 0) return launch_code<LPB, CP, Q, ODD, true>(a, code, teams, st);
  else if (long_words(a)) return launch_code<LPB, CP, Q, ODD, true>(a, code, teams, st);
  else return launch_code<LPB, CP, Q, ODD, false>(a, code, teams, st);
}

}  // namespace

// Lanes per bucket: one run of eight values (four up to d = 64) per lane up to d = 512, several
// runs of all 64 lanes beyond.  (Two runs per lane and half the lanes per bucket at d = 512
// share the work per bucket, but cost wavefronts: 53.7 us instead of 53.2 on 25.6M values,
// 42.4 instead of 41.3 on 20M sparser ones.)  Four runs of eight stay in registers for 1536 < d <=
// 2048, although that leaves two to four wavefronts per SIMD: reading them twice instead takes 20M
// values, s = 16, d = 1800 50.1 -> 58.7 us, Code'_s 46.5 -> 52.8, d = 2048 47.6 -> 49.5.  Few buckets: runs of four and twice the lanes
// up to d = 256, for the shortest chain.
static int lanes_per_bucket(uint32_t d, bool few) {
  if (d <= 64) return 16;
  if (d <= 128) return few ? 32 : 16;
  if (d <= 256) return few ? 64 : 32;
  return 64;
}
uint32_t direct_buckets_per_pass(uint32_t d, bool few) {
  return 64u / lanes_per_bucket(d, few && d % 4 == 0);
}

hipError_t launch_encode_direct(const EncodeArgs& a, uint32_t code, bool few, uint32_t teams,
                                hipStream_t st) {
  if (a.d % 4) {
    if (a.d <= 64) return launch_direct<16, 1, 1, true>(a, code, teams, st);
    if (a.d <= 128) return launch_direct<16, 1, 2, true>(a, code, teams, st);
    if (a.d <= 256) return launch_direct<32, 1, 2, true>(a, code, teams, st);
    if (a.d <= 512) return launch_direct<64, 1, 2, true>(a, code, teams, st);
    if (a.d <= 1024) return launch_direct<64, 2, 2, true>(a, code, teams, st);
    if (a.d <= 2048) return launch_direct<64, 4, 2, true>(a, code, teams, st);
    return launch_direct<64, 0, 2, true>(a, code, teams, st);
  }
  if (a.d <= 64) return launch_direct<16, 1, 1>(a, code, teams, st);
  if (a.d <= 128) return few ? launch_direct<32, 1, 1>(a, code, teams, st)
                             : launch_direct<16, 1, 2>(a, code, teams, st);
  if (a.d <= 256) return few ? launch_direct<64, 1, 1>(a, code, teams, st)
                             : launch_direct<32, 1, 2>(a, code, teams, st);
  if (a.d <= 512) return launch_direct<64, 1, 2>(a, code, teams, st);
  if (a.d <= 768) return launch_direct<64, 3, 1>(a, code, teams, st);
  if (a.d <= 1024) return launch_direct<64, 2, 2>(a, code, teams, st);
  if (a.d <= 1536) return launch_direct<64, 3, 2>(a, code, teams, st);
  if (a.d <= 2048) return launch_direct<64, 4, 2>(a, code, teams, st);
  return launch_direct<64, 0, 2>(a, code, teams, st);
}

}  // namespace qsgd
