// gfx950 (MI355X) kernels for paged-KV GQA attention: the device-side work
// planner, the persistent attention kernel (prefill-append tiles on bf16 MFMA and split-context
// decode items in one grid), and the split merge.
//
// The computation: new tokens of each sequence attend causally within their chunk and fully to
// the cached context (paper, Background: context growth p_{t+1} = p_t + r_t + o_t; Motivation:
// prefix caching and chunked prefill batched with decode; section 4.3, Eq. 1: decode cost per
// sequence is its KV-cache read).  Scores are s_j = scale * q.k_j over keys j <= position; the
// softmax is evaluated online in base 2 (exp(x) = 2^(x log2 e)), fp32 state, bf16 operands.
// The row sum l accumulates the fp32 weights (so the LSE is accurate to fp32); the weights enter
// the P.V product rounded to bf16 (round to nearest even).
//
// MFMA lane layouts used below (gfx950, bf16, fp32 accumulate; lane l of a 64-lane wave):
//   32x32x16: A row l%32, k 8*(l/32)+e;  B col l%32, k 8*(l/32)+e;
//             D col l%32, row (r%4) + 8*(r/4) + 4*(l/32) for accumulator r = 0..15.
//   16x16x32: A row l%16, k 8*(l/16)+e;  B col l%16, k 8*(l/16)+e;
//             D col l%16, row 4*(l/16) + r for r = 0..3.
// The contraction index k may be any permutation of the reduced dimension as long as A and B
// use the same one; the P.V products below use that freedom so the probabilities feed the B
// operand straight from the score accumulators.
//
// LDS transpose read (ds_read_b64_tr_b16): inside each 16-lane group, lane j supplies the
// address of an 8-byte row; lane l receives element l%4 of the rows supplied by lanes l/4,
// l/4+4, l/4+8, l/4+12.  With lane j addressing V[kbase + j/4][dbase + 4*(j%4)] (V row-major,
// keys x dims), lane l receives V[kbase + i][dbase + l%16] for i = 0..3: four consecutive keys
// of one dim, i.e. a k-contiguous MFMA operand of V^T.

#include "pearl_internal.h"

#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>
#include <mutex>

namespace pearl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define LDS_AS __attribute__((address_space(3)))

constexpr float kLn2 = 0.69314718055994530942f;

__device__ __forceinline__ u32x4 ld16(const uint16_t* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x8 zero_bf16x8() { return as_bf16x8(u32x4{0u, 0u, 0u, 0u}); }

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The XCD this wave runs on (hardware register XCC_ID, bits 3:0), in [0, kNumXcd).
__device__ __forceinline__ int xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) % kNumXcd; }
__device__ __forceinline__ float flog2(float x) { return __builtin_amdgcn_logf(x); }

__device__ __forceinline__ uint16_t bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__device__ __forceinline__ i16x4 lds_read_tr(const char* base, int byte_off) {
  // generic -> LDS address-space cast (the pointer always points into __shared__ memory)
  LDS_AS i16x4* p = (LDS_AS i16x4*)((LDS_AS char*)(base) + byte_off);
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p);
}

__device__ __forceinline__ bf16x8 concat_tr(i16x4 a, i16x4 b) {
  typedef short i16x8 __attribute__((ext_vector_type(8)));
  i16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// Combine x with the value held by lane l ^ 32, using v_permlane32_swap (one VALU instruction,
// no LDS round trip).  With both operands x, the swap returns r0 = (x[l] for l < 32, x[l-32]
// otherwise) and r1 = (x[l+32] for l < 32, x[l] otherwise); both halves then combine the same
// two values in the same order, so the results are bit-identical across the pair.
__device__ __forceinline__ float xor32_max(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}

__device__ __forceinline__ float xor32_add(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// The block table is read-only for the whole kernel; reading it through the constant address
// space lets the compiler use scalar loads (counted by lgkmcnt, not vmcnt) for these uniform reads.
typedef const __attribute__((address_space(4))) int32_t* ConstI32Ptr;

__device__ __forceinline__ int clamp_page(int p, int num_pages) {
  return p < 0 ? 0 : (p >= num_pages ? num_pages - 1 : p);
}

// The online softmax lets the running maximum m of a row lag the true maximum by up to kMaxLag
// (log2 units): weights 2^(s c - m) then stay below 2^kMaxLag, which bf16 and the fp32 sums hold
// as precisely as weights below 1.  A lane's 32 weights of a prefill stage summing to at most
// kMaxWeightSum guarantees that bound without finding the stage's maximum.
constexpr float kMaxLag = 8.0f;
constexpr float kMaxWeightSum = 256.0f;             // 2^kMaxLag

// LDS of the attention kernel beyond its separate arrays.  NW = waves per workgroup; kinds as
// in attn_kernel.
template <int D, int NW, int kKinds> struct Lds {
  // prefill stages travel by LDS-DMA into six stage buffers (three K, three V): separate arrays
  // in prefill-only kernels, carved from the region of the decode stages in the mixed kernel
  static constexpr int prefill_bytes = (kKinds == 3) ? 6 * kKeysPerStage * D * 2 : 0;
  static constexpr int decode_stage_bytes = NW * 2 * (2 * kPage * D * 2);   // per-wave K+V double buffer
  static constexpr int merge_bytes = NW * 8 * D * 4 + 2 * NW * 8 * 4;
  // decode-only kernels keep their stages in separate arrays; the mixed kernel carves them here
  static constexpr int decode_bytes = (kKinds == 3) ? decode_stage_bytes : 0;
  static constexpr int bytes0 = prefill_bytes > decode_bytes ? prefill_bytes : decode_bytes;
  static constexpr int bytes = bytes0 > 16 ? bytes0 : 16;
};

// ------------------------------------------------------------------------------------------------
// Planner: one workgroup validates the device-resident lengths against the host bounds and
// builds the work list (prefill q-tiles, then decode page-range splits), so no host sync is
// needed.  Writes the header, per-sequence records and entries; zeroes the work counters.
//
// Prefill tiles are split along the keys when the launch has too few of them to fill the compute
// units evenly.  All tiles of a sequence are cut at the same keys, multiples of its split_keys (the
// record's kind field holds split_keys / kKeysPerStage), the last split running to the tile's end;
// splits start at or before the first key that only some rows of the tile see (key ctx + t0 + 1),
// so every row sees at least one key of every split.
//   * Prefill launches of up to kPreSplitItems tile items: split_keys is the sequence's longest
//     tile cut into equal parts of at most P stages, P being 0.6, 0.75, 1 or 1.5 of the launch's
//     average stages per compute unit, whichever is the smallest whose splits fit the workspace's
//     partial slots.  Longest first, two or three splits per unit end together; one split of the
//     average length per unit leaves a second round of remainders: four turns of 91-392 tokens on
//     14-23K contexts (176 items) took 367 stages on the busiest unit for an average of 228, and
//     take 248 so (append, plan, attention and merge: 672 -> 459 us).  With more items than
//     kPreSplitItems whole tiles balance as well.
//   * Mixed launches of up to one tile item per compute unit whose longest tile would outlast the
//     average work per unit: split_keys is that average, at least kMinSplitKeys.  Work is estimated
//     in key-units: a prefill tile key (256 q-rows on MFMA) costs about 3/2 of a decode key (one
//     K/V row read from HBM).
//
// Prefill entries go longest first, in size classes, so the last entries a launch hands out are its
// shortest ones; inside a class the tiles that read the same keys follow one another, so they run
// at about the same time and share the caches.
//
// Decode splits hold pps pages each (the last one of a sequence the rest): pps is sized from the
// launch's actual pages (about kDecItemsPerCU items per compute unit) but never below the host's
// bound, so the workspace always holds the splits.  They are ordered longest first: every full
// split, then the shorter last splits in kPartBuckets size classes, largest class first, so the
// last items a launch hands out are its shortest ones.
//
// The kernel is latency from end to end (a first read of the lengths, then a few barriers, and the
// instruction fetches of code that runs once), so loops are not unrolled.
// ------------------------------------------------------------------------------------------------
constexpr int kPlanThreads = 256;
constexpr int kPlanWaves = kPlanThreads / 64;
constexpr int kPartBuckets = 16;
constexpr int kPreCandidates = 4;
constexpr int kPlanKeep = 4;               // prefill entries a thread keeps between the planner's rounds

// Size class of a short last split of `rest` pages (1 <= rest < pps); class 0 holds the longest.
// inv_pps = kPartBuckets / pps; the class only orders work, so rounding at a class edge is harmless.
__device__ __forceinline__ int part_bucket(int rest, float inv_pps) {
  return kPartBuckets - 1 - min(kPartBuckets - 1, (int)((float)(rest - 1) * inv_pps));
}

__device__ __forceinline__ int tile_splits(int ctx, int t0, int split_keys) {
  return split_keys > 0 ? (ctx + t0 + split_keys) / split_keys : 1;   // ceil((ctx + t0 + 1) / S)
}

__device__ __forceinline__ int key_stages(int keys) { return (keys + kKeysPerStage - 1) / kKeysPerStage; }

// split_keys of a sequence whose longest tile holds `stages` stages, for splits of at most P stages
// (0: whole tiles).
__device__ __forceinline__ int seq_split_keys(int stages, int P) {
  if (P <= 0 || stages <= P) return 0;
  const int ns = (stages + P - 1) / P;
  return (stages + ns - 1) / ns * kKeysPerStage;
}

struct PlanSeq { int ctx, q_len, split_keys; };

// kMode: kModePrefill, kModeDecode or kModeMixed.
template <int kMode>
__global__ __launch_bounds__(kPlanThreads) void plan_kernel(
    PlanParams p, const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu,
    int32_t* __restrict__ hdr, SeqInfo* __restrict__ seqinfo, int32_t* __restrict__ split_base,
    int2* __restrict__ entries, int4* __restrict__ pre_jobs) {
  __shared__ unsigned long long s_sum[2][kPlanWaves];      // prefill key-units, decode keys
  __shared__ int s_pages[kPlanWaves];                      // decode pages
  __shared__ int s_tiles[kPlanWaves], s_longest[kPlanWaves], s_bad[kPlanWaves];
  __shared__ int s_fits[kPreCandidates];                   // of each candidate P
  __shared__ int s_wave[4][kPlanWaves];
  __shared__ int s_part_cnt[kPartBuckets], s_part_off[kPartBuckets];   // short last decode splits
  __shared__ int s_tile_cnt[kPartBuckets], s_tile_off[kPartBuckets];   // prefill entries
  __shared__ int s_jobs;
  __shared__ PlanSeq s_seq[kPlanThreads];                  // a chunk's prefill sequences
  __shared__ int s_pre[kPlanThreads + 1];                  // prefix sums of their candidate entries
  __shared__ int s_slot[kPlanThreads];                     // their first partial slots
  __shared__ SeqInfo s_first[kPlanThreads];                // the first chunk's sequences
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = p.tokens_per_tile, H = p.num_kv_heads;
  // counts scanned per sequence: decode splits, full decode splits, candidate prefill entries, slots
  constexpr int C0 = kMode == kModePrefill ? 2 : 0, C1 = kMode == kModeDecode ? 2 : 4;
  const int log_t = __builtin_ctz(T);               // T is a power of two
  auto tiles_of = [&](int q_len) { return (q_len + T - 1) >> log_t; };
  const int chunks = (p.batch + kPlanThreads - 1) / kPlanThreads;
  if (tid < kPartBuckets) { s_part_cnt[tid] = 0; s_tile_cnt[tid] = 0; }
  if (tid == 0) s_jobs = 0;
  if (tid < kHdrWords - kHdrZero) hdr[kHdrZero + tid] = 0;   // zero block read by decode items
  if (tid < kNumXcd) hdr[kHdrQueues + tid] = 0;
  // sequence b's lengths
  auto seq_of = [&](int b) {
    SeqInfo s{b, 1, ctx_lens[b], kSeqNone};
    if (cu) {
      s.q_start = cu[b];
      s.q_len = cu[b + 1] - s.q_start;
    }
    if (s.q_len > 0)
      s.kind = kMode == kModeDecode || (kMode == kModeMixed && s.q_len == 1) ? kSeqDecode : kSeqPrefill;
    return s;
  };
  // pass 1: validate every sequence and total the work
  SeqInfo mine{0, 0, 0, kSeqNone};                  // of the first chunk
  {
    int tiles = 0, longest = 0, dpages = 0;         // pages: batch * bt_stride fits 32 bits
    unsigned long long sum[2] = {0, 0};
    bool bad = false;
#pragma unroll 1
    for (int b = tid; b < p.batch; b += kPlanThreads) {
      const SeqInfo s = seq_of(b);
      if (b == tid) s_first[tid] = mine = s;
      const long long kv = (long long)s.ctx_len + s.q_len;
      if (s.q_len < 0 || s.ctx_len < 0 || s.q_start < 0 || s.q_len > p.max_q_len ||
          (long long)s.q_start + s.q_len > p.total_q || kv > p.max_kv_len || (kv + kPage - 1) / kPage > p.bt_stride ||
          (kMode == kModeDecode && s.q_len != 1)) {
        bad = true;
      } else if (kMode != kModePrefill && s.kind == kSeqDecode) {
        sum[1] += (unsigned long long)kv;
        dpages += (int)((kv + kPage - 1) / kPage);
      } else if (kMode != kModeDecode && s.kind == kSeqPrefill) {
        const int nt = tiles_of(s.q_len);
        tiles += nt;
        // keys seen by every row of tile t: ctx + t T + 1
        sum[0] += (unsigned long long)nt * (s.ctx_len + 1) + (unsigned long long)T * nt * (nt - 1) / 2;
        longest = max(longest, (int)kv);
      }
    }
#pragma unroll 1
    for (int off = 32; off >= 1; off >>= 1) {
      if (kMode != kModeDecode) {
        tiles += __shfl_xor(tiles, off);
        longest = max(longest, __shfl_xor(longest, off));
        sum[0] += __shfl_xor(sum[0], off);
      }
      if (kMode != kModePrefill) {
        sum[1] += __shfl_xor(sum[1], off);
        dpages += __shfl_xor(dpages, off);
      }
    }
    const bool wave_bad = __any(bad);
    if (lane == 0) {
      s_tiles[wv] = tiles;
      s_longest[wv] = longest;
      s_bad[wv] = wave_bad;
      s_sum[0][wv] = sum[0];
      s_sum[1][wv] = sum[1];
      s_pages[wv] = dpages;
    }
  }
  __syncthreads();
  int tiles = 0, longest = 0, bad = 0;
  unsigned long long pre_keys = 0, dec_keys = 0, dec_pages = 0;
#pragma unroll
  for (int w = 0; w < kPlanWaves; ++w) {
    tiles += s_tiles[w];
    longest = max(longest, s_longest[w]);
    bad |= s_bad[w];
    pre_keys += s_sum[0][w];
    dec_keys += s_sum[1][w];
    dec_pages += s_pages[w];
  }
  if (bad) {
    if (tid == 0) {
      hdr[kHdrCounter] = 0; hdr[kHdrNumPre] = 0; hdr[kHdrNumDec] = 0; hdr[kHdrPreFirstWG] = 0;
      hdr[kHdrError] = 1; hdr[kHdrNumItems] = 0; hdr[kHdrPreSplitKeys] = 0; hdr[kHdrNumPreJobs] = 0;
      hdr[kHdrPagesPerSplit] = p.pages_per_split;
    }
    return;
  }
  // Prefill splits: the first of the candidates whose entries and partial slots fit.  P: the most
  // stages of a split (prefill launches); mixed_keys: split_keys of every sequence (mixed ones).
  const long long pre_units = (long long)pre_keys * H;
  int P = 0, mixed_keys = 0;
  constexpr bool is_mixed = kMode == kModeMixed;
  if (kMode != kModeDecode && p.pre_slots > 0 && tiles > 0 && (long long)tiles * H <= (is_mixed ? kPlanComputeUnits : kPreSplitItems)) {
    const long long work = pre_units + pre_units / 2 + (long long)dec_keys * H;
    const long long per_cu = (work + kPlanComputeUnits - 1) / kPlanComputeUnits;
    const long long share_keys = (pre_units + kPlanComputeUnits - 1) / kPlanComputeUnits;
    const int share = (int)((share_keys + kKeysPerStage - 1) / kKeysPerStage);
    const int S0 = max(kMinSplitKeys / kKeysPerStage,
                       max(share, (int)(((2 * per_cu + 2) / 3 + kKeysPerStage - 1) / kKeysPerStage)));
    constexpr int kLeast = kMinSplitKeys / kKeysPerStage;
    auto cand = [&](int c) {                        // stages
      if (is_mixed) return S0 << c;
      return c == 0 ? max(kLeast / 2, (3 * share + 4) / 5)
                    : c == 1 ? max(kLeast / 2, (3 * share + 3) / 4) : max(kLeast, c == 2 ? share : share + share / 2);
    };
    static_assert(kPlanWaves == kPreCandidates, "a wave per candidate");
    const int my_cand = cand(wv);
    int n_entries = 0, n_slots = 0;
#pragma unroll 1
    for (int b = lane; b < p.batch; b += 64) {
      const SeqInfo s = b < kPlanThreads ? s_first[b] : seq_of(b);
      if (s.kind != kSeqPrefill) continue;
      const int nt = tiles_of(s.q_len);
      const int S = is_mixed ? my_cand * kKeysPerStage : seq_split_keys(key_stages(s.ctx_len + s.q_len), my_cand);
      const int n = nt * tile_splits(s.ctx_len, (nt - 1) * T, S);
      n_entries += n;
      if (S > 0) n_slots += n;
    }
#pragma unroll 1
    for (int off = 32; off >= 1; off >>= 1) {
      n_entries += __shfl_xor(n_entries, off);
      n_slots += __shfl_xor(n_slots, off);
    }
    if (lane == 0) s_fits[wv] = n_entries <= p.max_pre && (long long)n_slots * H <= p.pre_slots && n_slots <= p.pre_jobs_cap;
    __syncthreads();
#pragma unroll
    for (int c = kPreCandidates - 1; c >= 0; --c)
      if (s_fits[c]) P = cand(c);
    if (P >= key_stages(longest)) P = 0;            // no tile would split
    if (is_mixed) {
      mixed_keys = P * kKeysPerStage;
      P = 0;
    }
  }
  auto split_of = [&](const SeqInfo& s) {
    return mixed_keys > 0 ? mixed_keys : seq_split_keys(key_stages(s.ctx_len + s.q_len), P);
  };
  // Decode split size: about kDecItemsPerCU items per compute unit over the launch's actual
  // pages, a multiple of 16 pages, at least the host's bound and at most kMaxPagesPerSplit.
  // Splits of at least kDecLongSplitPages pages (16 pages per wave) while that still leaves
  // 2 items per compute unit: a wave's first page of an item waits unhidden, so short splits
  // pay it often.
  int pps = p.pages_per_split;
  if (kMode != kModePrefill && dec_pages > 0) {
    const unsigned long long units = dec_pages * H;
    const unsigned long long per = (unsigned long long)kPlanComputeUnits * kDecItemsPerCU;
    const unsigned long long want = (units + per - 1) / per, two = (units + 2 * kPlanComputeUnits - 1) / (2 * kPlanComputeUnits);
    const unsigned long long top = max(p.pages_per_split, kMaxPagesPerSplit);
    pps = max(pps, (int)min(top, (want + 15) / 16 * 16));
    pps = max(pps, (int)min((unsigned long long)kDecLongSplitPages, (two + 15) / 16 * 16));
  }
  const float inv_pps = (float)kPartBuckets / (float)pps;
  // size classes of prefill entries, by their stages; the longest possible entry is in class 0
  const int max_stages = mixed_keys > 0 ? mixed_keys / kKeysPerStage : (P > 0 ? P : key_stages(longest));
  const float inv_stages = (float)kPartBuckets / (float)(max_stages + 1);
  // The sequences, a chunk at a time: round 0 counts the classes, round 1 writes the records and the
  // entries.  Usually there is one chunk and each thread has at most kPlanKeep prefill entries: it
  // keeps what round 0 found (class and rank in it), and round 1 only writes.
  int carry[4] = {0, 0, 0, 0};
  int keep_pos[kPlanKeep], keep_code[kPlanKeep], keep_seq[kPlanKeep];
  bool keeps = false;
  int cnt[4], excl[4] = {0, 0, 0, 0}, total[4] = {0, 0, 0, 0}, rest = 0, split_keys = 0, part_class = 0, part_rank = 0;
  SeqInfo s = mine;
  auto keeps_now = [&](int chunk, int entries_) { return chunk == 0 && chunks == 1 && entries_ <= kPlanKeep * kPlanThreads; };
#pragma unroll 1
  for (int round = 0; round < 2; ++round) {
    if (!keeps) {
#pragma unroll
      for (int c = 0; c < 4; ++c) carry[c] = 0;
    }
#pragma unroll 1
    for (int chunk = 0; chunk < chunks; ++chunk) {
      const int b = chunk * kPlanThreads + tid;
      if (!keeps) {
        s = SeqInfo{0, 0, 0, kSeqNone};
        if (b < p.batch) s = chunk == 0 ? mine : seq_of(b);
        // decode splits, full decode splits, candidate prefill entries, partial slots
#pragma unroll
        for (int c = 0; c < 4; ++c) cnt[c] = 0;
        rest = split_keys = 0;
        if (kMode != kModePrefill && s.kind == kSeqDecode) {
          const int pages = (s.ctx_len + s.q_len + kPage - 1) / kPage;
          cnt[0] = (pages + pps - 1) / pps;
          cnt[1] = pages / pps;
          rest = pages - cnt[1] * pps;
        } else if (kMode != kModeDecode && s.kind == kSeqPrefill) {
          const int nt = tiles_of(s.q_len);
          split_keys = split_of(s);
          cnt[2] = nt * tile_splits(s.ctx_len, (nt - 1) * T, split_keys);
          cnt[3] = split_keys > 0 ? cnt[2] : 0;
        }
        // exclusive scan: wave-level inclusive scans by shuffles, then the totals of earlier waves
        int incl[4] = {cnt[0], cnt[1], cnt[2], cnt[3]};
#pragma unroll 1
        for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
          for (int c = C0; c < C1; ++c) {
            const int u = __shfl_up(incl[c], off);
            if (lane >= off) incl[c] += u;
          }
        }
        if (lane == 63) {
#pragma unroll
          for (int c = C0; c < C1; ++c) s_wave[c][wv] = incl[c];
        }
        if (rest) {
          part_class = part_bucket(rest, inv_pps);
          part_rank = atomicAdd(&s_part_cnt[part_class], 1);
        }
        __syncthreads();
#pragma unroll
        for (int c = C0; c < C1; ++c) {
          int before = 0;
          total[c] = 0;
#pragma unroll
          for (int w = 0; w < kPlanWaves; ++w) {
            if (w < wv) before += s_wave[c][w];
            total[c] += s_wave[c][w];
          }
          excl[c] = carry[c] + before + incl[c] - cnt[c];
        }
        s_seq[tid] = PlanSeq{s.ctx_len, s.q_len, split_keys};
        s_slot[tid] = excl[3];
        s_pre[tid + 1] = excl[2] - carry[2] + cnt[2];
        if (tid == 0) s_pre[0] = 0;
        __syncthreads();
      }
      if (round && b < p.batch) {
        seqinfo[b] = SeqInfo{s.q_start, s.q_len, s.ctx_len,
                             s.kind == kSeqPrefill ? kSeqPrefill | (split_keys / kKeysPerStage << 4) : s.kind | (cnt[0] << 4)};
        split_base[b] = s.kind == kSeqPrefill ? excl[3] : excl[0];
        // full splits in sequence order, the short last split at its size class's next position
        const int part_pos = rest ? s_part_off[part_class] + part_rank : 0;
#pragma unroll 1
        for (int sp = 0; sp < cnt[0]; ++sp) {
          const int pos = sp < cnt[1] ? excl[1] + sp : part_pos;
          if (pos < p.max_dec) entries[p.max_pre + pos] = make_int2(b, sp);
        }
      }
      // Prefill entries, a thread each: (split, tile) of a sequence, the tile running fastest, last
      // tile first.  Returns the entry's class and rank, or -1 if there is none (shorter tiles of a
      // sequence have fewer splits).
      auto find = [&](int i, int& lo, int& code, int& rank) {
        lo = 0;
        int hi = min(kPlanThreads, p.batch - chunk * kPlanThreads) - 1;
        while (lo < hi) {                           // the last sequence whose entries start at or before i
          const int mid = (lo + hi + 1) >> 1;
          if (s_pre[mid] <= i) lo = mid; else hi = mid - 1;
        }
        const PlanSeq q = s_seq[lo];
        const int nt = tiles_of(q.q_len), j = i - s_pre[lo];
        const int sp = j / nt, t = nt - 1 - (j - sp * nt);
        const int ns = tile_splits(q.ctx, t * T, q.split_keys);
        if (sp >= ns) return -1;
        const int step = q.split_keys / kKeysPerStage;
        const int stages = sp + 1 < ns ? step : key_stages(q.ctx + min(q.q_len, (t + 1) * T)) - sp * step;
        const int k = kPartBuckets - 1 - min(kPartBuckets - 1, (int)((float)stages * inv_stages));
        code = t | (sp << 16);
        rank = atomicAdd(&s_tile_cnt[k], 1);
        if (round == (keeps_now(chunk, total[2]) ? 0 : 1) && sp == 0 && ns > 1) {
          const int job = atomicAdd(&s_jobs, 1);
          if (job < p.pre_jobs_cap) pre_jobs[job] = make_int4(chunk * kPlanThreads + lo, t, s_slot[lo] + t, ns);
        }
        return k;
      };
      if (!keeps && keeps_now(chunk, total[2])) {
#pragma unroll
        for (int u = 0; u < kPlanKeep; ++u) {
          keep_pos[u] = -1;
          const int i = tid + u * kPlanThreads;
          if (i < total[2]) {
            int rank = 0;
            const int k = find(i, keep_seq[u], keep_code[u], rank);
            if (k >= 0) keep_pos[u] = k << 24 | rank;
          }
        }
      } else if (keeps) {
#pragma unroll
        for (int u = 0; u < kPlanKeep; ++u) {
          if (keep_pos[u] < 0) continue;
          const int pos = s_tile_off[keep_pos[u] >> 24] + (keep_pos[u] & 0xffffff);
          if (pos < p.max_pre) entries[pos] = make_int2(keep_seq[u], keep_code[u]);
        }
      } else {
#pragma unroll 1
        for (int i = tid; i < total[2]; i += kPlanThreads) {
          int lo, code = 0, rank = 0;
          const int k = find(i, lo, code, rank);
          if (!round || k < 0) continue;
          const int pos = s_tile_off[k] + rank;
          if (pos < p.max_pre) entries[pos] = make_int2(chunk * kPlanThreads + lo, code);
        }
      }
      if (!keeps) {
        __syncthreads();
#pragma unroll
        for (int c = C0; c < C1; ++c) carry[c] += total[c];
      }
    }
    if (round == 0) {
      // offsets of the classes, largest first (decode: after the full splits)
      if (tid < kPartBuckets) {
        int off = carry[1], toff = 0;
#pragma unroll
        for (int k = 0; k < kPartBuckets; ++k) {    // all reads in flight together
          const int c = s_part_cnt[k], t = s_tile_cnt[k];
          if (k < tid) { off += c; toff += t; }
        }
        s_part_off[tid] = off;
        s_tile_off[tid] = toff;
      }
      keeps = keeps_now(0, total[2]);
      __syncthreads();
      if (!keeps) {
        if (tid < kPartBuckets) { s_part_cnt[tid] = 0; s_tile_cnt[tid] = 0; }   // now the fill counts
        __syncthreads();
      }
    }
  }
  if (tid == 0) {
    const int n_pre = s_tile_off[kPartBuckets - 1] + s_tile_cnt[kPartBuckets - 1];
    const int n_dec = carry[0], n_jobs = s_jobs;
    const bool over = n_pre > p.max_pre || n_dec > p.max_dec || n_jobs > p.pre_jobs_cap ||
                      (long long)carry[3] * H > p.pre_slots;
    // Mixed launches: how many workgroups take prefill items first (the others take decode items
    // first): 1.2 x prefill's share of the estimated work, in prefill and decode key-units
    // weighted 3 : 2 as above.  A prefill tile left for the end of a launch holds one workgroup
    // far longer than a decode split, so prefill gets more than its share.
    if (kMode == kModeMixed) {
      const double pu = 3.0 * (double)pre_units, du = 2.0 * (double)((long long)dec_keys * H);
      hdr[kHdrPreFirstWG] = pu + du > 0 ? (int)fmin((double)p.mixed_grid, 1.2 * p.mixed_grid * pu / (pu + du)) : p.mixed_grid;
    }
    hdr[kHdrCounter] = 0;
    hdr[kHdrNumPre] = over ? 0 : n_pre;
    hdr[kHdrNumDec] = over ? 0 : n_dec;
    hdr[kHdrError] = over ? 2 : 0;
    hdr[kHdrNumItems] = over ? 0 : (n_pre + n_dec) * H;
    hdr[kHdrPreSplitKeys] = mixed_keys > 0 ? mixed_keys : P * kKeysPerStage;
    hdr[kHdrNumPreJobs] = over ? 0 : n_jobs;
    hdr[kHdrPagesPerSplit] = pps;
  }
}

// 16 bytes per lane from global memory straight into LDS (lane l writes lds_base + 16 l), issued
// as inline assembly, which the compiler does not track: it then inserts no waits of its own for
// it (it would wait for every copy in flight before any LDS read), and the caller waits with
// explicit vmcnt counts.  The compiler's own vmcnt waits stay correct, because copies it does
// not know about can only make them wait longer.  The LDS base goes through M0, which the
// sequence saves and restores (the copy reads it at issue, one wait state after it is written).
// lds_base must be uniform across the wave.  kOnce: the load is marked non-temporal (nt), for
// bytes read once per launch.
template <bool kOnce = false>
__device__ __forceinline__ void lds_dma16_untracked(const void* g, const char* lds_base) {
  const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)((LDS_AS const char*)lds_base));
  unsigned saved;
  if constexpr (kOnce) {
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off nt\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(g), "s"(lds)
        : "memory");
  } else {
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(g), "s"(lds)
        : "memory");
  }
}

// The same for rows that follow one another in memory and in LDS, from a uniform base and 32-bit lane
// offsets: N instructions, 1 KiB further each in both (the immediate offset advances the source and
// the LDS address alike).  A wave is held until the address unit has taken each copy, and copies of
// 64-bit lane addresses held it longer, besides the vector adds that formed them: 16 chunks of
// 256-2048 tokens on 5-24K contexts (MFMA-bound) took 4080 us with those and take 3850 with these
// (1.13 -> 1.20 PF/s), four turns 467 -> 446, the colocated batch 1338 -> 1280 with its decode pages
// copied this way too.
template <int N>
__device__ __forceinline__ void lds_dma16_rows(const char* base, const int* off, const char* lds_base) {
  static_assert(N == 1 || N == 2, "rows");
  const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)((LDS_AS const char*)lds_base));
  unsigned saved;
  if constexpr (N == 2)
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %4\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %3\n\t"
        "global_load_lds_dwordx4 %2, %3 offset:1024\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(off[0]), "v"(off[N - 1]), "s"(base), "s"(lds)
        : "memory");
  else
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(off[0]), "s"(base), "s"(lds)
        : "memory");
}

// vmcnt(n) with the other counters left alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
#define PEARL_VMCNT(n) (((n) & 15) | (((n) >> 4) << 14) | 0x0F70)
// lgkmcnt(0) with the other counters left alone
#define PEARL_LGKMCNT0 0xC07F

// A prefill stage staged by LDS-DMA: kKeysPerStage key rows of D bf16, unpadded.  The 16-byte
// chunk q of row r sits in slot q ^ swz(r), which keeps both operand read patterns free of bank
// conflicts on the 64 banks of 4 bytes: the row reads of the Q.K products (16 lanes read one chunk
// of 16 consecutive rows: swz is a permutation of the 16 rows' slots) and the transposing reads of
// the P.V products (32 lanes read 4 adjacent chunks of 4 consecutive rows: swz moves each of the 4
// rows to its own quarter of the 256 bank bytes).  Wave w copies rows [RPW w, RPW w + RPW) of the
// stage, RPI rows per 64-lane DMA instruction.
template <int D, int KEYS = kKeysPerStage> struct DmaTile {
  static_assert(D == 64 || D == 128, "head_dim");
  static constexpr int CPR = D / 8;                 // 16-byte chunks per row
  static constexpr int RB = D * 2;                  // bytes per row
  static constexpr int BYTES = KEYS * RB;
  static constexpr int RPI = 64 / CPR;              // rows per DMA instruction
  static constexpr int RPW = KEYS / kWaves;         // rows copied per wave
  static constexpr int NDMA = RPW / RPI;            // DMA instructions per wave and tensor
  static_assert(NDMA >= 1 && NDMA * RPI == RPW && kPage % RPW == 0, "DMA split");
  __device__ static __forceinline__ int swz(int r) {
    // d = 128: a row is all 64 banks, rows 4i..4i+3 get slot offsets 0, 4, 8, 12 (+ i);
    // d = 64: two rows share the banks, rows 4i..4i+3 get offsets 0, 0, 4, 4 (+ i)
    if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
    else return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
  }
};

// ------------------------------------------------------------------------------------------------
// Prefill-append work item: one (sequence, kv-head g, q-tile).  The tile holds 256 q-rows =
// tokens_per_tile tokens x G heads of the group (row rho -> token rho / G, head rho % G), so every
// staged K/V byte is shared by the whole group.  Wave w owns rows [32w, 32w+32).
//   S^T (keys x rows) = K . Q^T     (32x32x16 MFMA: A = K tile from LDS, B = Q^T in registers)
//   O^T (dims x rows) += V^T . P^T  (A = V^T via LDS transpose reads, B = P^T from S^T registers)
// Each lane owns one q-row (l%32) for both products, so the softmax row statistics are
// lane-local apart from one exchange with lane l^32, which holds the row's other keys.
// A split item (code = tile | split << 16) covers only its key range and writes the unnormalised
// (o~, m, l) of its rows to partial slot (base + split * tiles + tile) * H_kv + g, base being its
// sequence's split_base, for the prefill merge.
//
// Schedule (prefill-only and mixed kernels): the matrix and vector work of the two waves on each
// SIMD overlap.  The 8 waves form two groups, waves 0-3 and waves 4-7 (the waves w and w + 4 share
// a SIMD), and the item runs in phases separated by workgroup barriers.  In each of its phases a
// wave does either
//   M(j): S(j) = K(j) Q^T and O += V(j-1)^T P(j-1)   (32 MFMAs at d = 128, no dependence between
//         the two products), or
//   V(j): the online softmax of S(j), giving P(j)    (exp, scale and sums on the vector ALU),
// alternating M(0) V(0) M(1) V(1) ... M(n); group B runs one phase behind group A.  In every phase
// one wave of each SIMD therefore issues MFMAs while the other runs its softmax, so the matrix core
// works through the vector phase of the other wave instead of waiting for it.
// Stages travel by LDS-DMA into three DmaTile buffers per tensor: K(j) into K buffer j % 3, V(j)
// into V buffer j % 3.  K(j) is
// read in phases 2j and 2j+1, V(j) in phases 2j+2 and 2j+3.  Each wave copies its rows of K(j+2)
// and V(j+1) (the pair j) in phases 2j and 2j+1, into buffers last read in phase 2j-1: half of the
// DMA instructions right after its MFMAs of M(j), the other half at the start of its adjacent
// softmax phase.  A DMA instruction holds its wave for tens of cycles before it is accepted, and
// longer when many queue at the compute unit at once: issued all together at a phase start they
// stalled every wave for hundreds of cycles; after the MFMAs they overlap the draining matrix
// pipeline, and at the start of a softmax phase they use the slack that phase has over an M phase.
// Before the barrier that ends phase 2j-1 every wave waits for its own copies of K(j) and V(j-1)
// (the copies issued since stay in flight).
// ------------------------------------------------------------------------------------------------
// at_end: called by every thread when the stages are done, before the epilogue.
template <int D, typename AtEnd>
__device__ __forceinline__ void prefill_tile_pp(const AttnArgs& a, int b, int code, int g, char* kb0, char* vb0, AtEnd at_end) {
  constexpr int KB = D / 16;                        // 16-wide k blocks of the QK product
  constexpr int MB = D / 32;                        // 32-wide dim blocks of the PV product
  constexpr int SK = kKeysPerStage;                 // keys per stage
  constexpr int NST = SK / 32;                      // 32-key sub-tiles per stage
  static_assert(kKeysPerStage % SK == 0, "key splits stay stage-aligned");
  using DT = DmaTile<D, SK>;
  constexpr int RB = DT::RB;
  // buffer r of each tensor (r = stage % 3 is a compile-time constant wherever a buffer is used, so
  // every LDS address is a per-lane offset plus an immediate)
  auto kbuf = [&](int r) { return kb0 + r * DT::BYTES; };
  auto vbuf = [&](int r) { return vb0 + r * DT::BYTES; };

  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index (uniform)
  const int grp = w >> 2;                           // 0: waves 0-3, 1: waves 4-7 (one phase later)
  const SeqInfo si = a.seqinfo[b];
  const int G = a.group;
  const int tile = code & 0xffff, split = code >> 16;
  const int t0 = tile * a.tokens_per_tile;
  const int t_end = min(t0 + a.tokens_per_tile, si.q_len);
  const int ctx = si.ctx_len;
  const int kv_needed = ctx + t_end;
  const int rho = 32 * w + (lane & 31);
  const int tok = t0 + rho / G;
  const int hh = rho - (rho / G) * G;
  const int h = g * G + hh;
  const bool row_ok = tok < t_end;
  const int row_limit = ctx + tok;                  // last visible key of this row
  const int wave_min_limit = ctx + t0 + (32 * w) / G;
  const int H_q = a.num_q_heads, H_kv = a.num_kv_heads;
  const size_t head_stride = (size_t)kPage * D;     // elements per (page, kv-head) block
  const float c = a.scale_log2;

  bf16x8 qop[KB];
  {
    const uint16_t* qrow = a.q + ((size_t)(si.q_start + (row_ok ? tok : t0)) * H_q + h) * D + 8 * half;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) qop[kb] = row_ok ? as_bf16x8(ld16(qrow + 16 * kb)) : zero_bf16x8();
  }
  f32x16 oacc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[mb][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const int n_steps = (kv_needed + SK - 1) / SK;
  const int split_keys = (si.kind >> 4) * kKeysPerStage;
  const int n_split = tile_splits(ctx, t0, split_keys);
  const int step_begin = split * (split_keys / SK);
  const int step_end = split + 1 < n_split ? step_begin + split_keys / SK : n_steps;
  const int n = step_end - step_begin;              // stages of this item (>= 1)

  const ConstI32Ptr bt_c = (ConstI32Ptr)(a.block_table + (size_t)b * a.bt_stride);
  const int last_pidx = (kv_needed - 1) / kPage;
  const int gi = lane >> 4, jl = lane & 15;
  const int krow = 4 * (gi >> 1) + (jl >> 2);
  const int dcol = 16 * (gi & 1) + 4 * (jl & 3);
  int koff[KB], voff[2][MB], goff[DT::NDMA];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) koff[kb] = (lane & 31) * RB + (((2 * kb + half) ^ DT::swz(lane & 15)) << 4);
#pragma unroll
  for (int sec = 0; sec < 2; ++sec)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = krow + 8 * sec;
      voff[sec][mb] = r * RB + ((((32 * mb + dcol) >> 3) ^ DT::swz(r)) << 4) + (jl & 1) * 8;
    }
#pragma unroll
  for (int i = 0; i < DT::NDMA; ++i) {
    const int r = DT::RPW * w + DT::RPI * i + lane / DT::CPR;
    goff[i] = (r % kPage) * RB + (((lane % DT::CPR) ^ DT::swz(r)) << 4) - i * 1024;   // less the immediate offset
  }
  // this wave's rows of the K (or V) tile of local stage j, by LDS-DMA; V rows past the last
  // needed key come from the workspace's zero block (K rows there are always masked)
  const char* zero_src = reinterpret_cast<const char*>(a.ws_hdr + kHdrZero);
  // block-table entry of this wave's rows of local stage j (a scalar load; clamped where used)
  auto page_of = [&](int j) {
    const int pidx = min(((step_begin + j) * SK + DT::RPW * w) / kPage, last_pidx);
    return bt_c[pidx];
  };
  // this wave's rows of local stage j; V rows past the last needed key can only be in its last stage
  auto dma = [&](int j, bool is_v, int entry, char* dst) {
    const int page = clamp_page(entry, a.num_pages);
    const size_t base = (((size_t)page * H_kv + g) * head_stride) * 2;
    const char* src = reinterpret_cast<const char*>(is_v ? a.v_pool : a.k_pool) + base;
    const int row0 = DT::RPW * w, key0 = (step_begin + j) * SK + row0;
    if (!is_v || key0 + DT::RPW <= kv_needed) {
      lds_dma16_rows<DT::NDMA>(src, goff, dst + row0 * RB);
    } else {
#pragma unroll
      for (int i = 0; i < DT::NDMA; ++i) {
        const int key = key0 + DT::RPI * i + lane / DT::CPR;
        lds_dma16_untracked(key >= kv_needed ? zero_src : src + goff[i] + i * 1024, dst + (row0 + DT::RPI * i) * RB);
      }
    }
  };

  // block-table entries of the next copies: pid_k for K rows, pid_v for V rows (pid_n: the K
  // rows after those, read ahead by group B)
  int pid_v = 1 < n ? page_of(1) : 0, pid_k = 2 < n ? page_of(2) : 0, pid_n = 0;

  f32x16 s[NST];                                    // S^T of the stage between its M and V phases
  bf16x8 pop[NST][2];                               // P^T of the stage between its V and next M phases
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < NST; ++st) s[st] = zero16;
#pragma unroll
  for (int st = 0; st < NST; ++st)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) pop[st][kk] = zero_bf16x8();

  // M(j): PV of stage j - 1 (if any), then QK of stage j (if any).  P(j - 1) dies before S(j) is
  // born, so the two share registers.  The phase is one wave's stream of MFMAs while the other
  // wave of its SIMD runs a softmax, so nothing else hides its LDS latency: the operands are read
  // kLead MFMAs ahead through a small ring, and a scheduling barrier after each step keeps that
  // order (the compiler would otherwise read each operand just before its MFMA).
  constexpr int NPV = 2 * NST * MB, NQK = NST * KB, kLead = 3;
  auto operand = [&](int i, const char* kb_, const char* vb_) -> bf16x8 {
    if (i < NPV) {                                  // V^T of (dim block, sub-tile, 16-key half)
      const int mb = i / (2 * NST), st = (i >> 1) % NST, kk = i & 1;
      const int vo = (32 * st + 16 * kk) * RB;
      return concat_tr(lds_read_tr(vb_, vo + voff[0][mb]), lds_read_tr(vb_, vo + voff[1][mb]));
    }
    const int q = i - NPV, st = q / KB, kb = q - (q / KB) * KB;   // K rows of (sub-tile, k block)
    return *reinterpret_cast<const bf16x8*>(kb_ + 32 * st * RB + koff[kb]);
  };
  auto mfma_slot = [&](int i, const bf16x8& op) {
    if (i < NPV) {
      const int mb = i / (2 * NST), st = (i >> 1) % NST, kk = i & 1;
      oacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, pop[st][kk], oacc[mb], 0, 0, 0);
    } else {
      const int q = i - NPV, st = q / KB, kb = q - (q / KB) * KB;
      s[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, qop[kb], kb == 0 ? zero16 : s[st], 0, 0, 0);
    }
  };
  constexpr int NM = NPV + NQK;
  // One instruction stream for every M phase (no joins of differently allocated copies): M(0)
  // adds P = 0 times a zero-filled V buffer 2, and M(n) computes an S that no V phase reads.
  // R = j % 3: K(j) sits in K buffer R and V(j - 1) in V buffer (R + 2) % 3.
  // The first kLead operands (V^T reads) of an M phase are read at the end of the softmax phase
  // before it, so that their latency passes while the wave waits at the barrier.
  bf16x8 ring[kLead];
  auto prefetch = [&](auto r_c) {
    constexpr int R = decltype(r_c)::value;
#pragma unroll
    for (int d = 0; d < kLead; ++d) ring[d] = operand(d, kbuf(R), vbuf((R + 2) % 3));
  };
  auto phase_m = [&](auto r_c, bool prefetched) {
    constexpr int R = decltype(r_c)::value;
    const char* kb_ = kbuf(R);
    const char* vb_ = vbuf((R + 2) % 3);
    if (!prefetched) prefetch(r_c);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const bf16x8 op = ring[i % kLead];
      if (i + kLead < NM) ring[i % kLead] = operand(i + kLead, kb_, vb_);
      mfma_slot(i, op);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // The copies of stage j's pair: K(j + 2) into K buffer (R + 2) % 3 and V(j + 1) into V buffer
  // (R + 1) % 3 (R = j % 3).
  auto copy_k = [&](auto r_c, int j) {
    constexpr int R = decltype(r_c)::value;
    if (j + 2 < n) dma(j + 2, false, pid_k, kbuf((R + 2) % 3));
  };
  auto copy_v = [&](auto r_c, int j) {
    constexpr int R = decltype(r_c)::value;
    if (j + 1 < n) dma(j + 1, true, pid_v, vbuf((R + 1) % 3));
  };
  // V(j), 0 <= j < n: causal mask (only on stages that reach past some row's last visible key; the
  // empty asm keeps that a real branch), then the online softmax (base 2).  The weights are first
  // taken against the running maximum m without looking for this stage's maximum; that is exact
  // (any m gives the same softmax) as long as no weight exceeds 2^kMaxLag, which the lane's sum of
  // its 32 weights bounds.  Otherwise (the first stage of an item, where m is still -inf, or
  // scores jumping more than kMaxLag above m) the stage is redone with the row maximum, and m
  // moves to it only when it exceeds m by more than kMaxLag, so the O rescale is rare too.  A NaN
  // sum (a masked key against m = -inf) also takes the redo.
  auto phase_v = [&](int j) {
    const int k0 = (step_begin + j) * SK;
    if (k0 + SK - 1 > wave_min_limit) {
      __asm__ volatile("" ::);
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + 32 * st + (r & 3) + 8 * (r >> 2) + 4 * half;
          if (key > row_limit) s[st][r] = -INFINITY;
        }
    }
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float pv = fexp2(__builtin_fmaf(s[st][r], c, -m_run));
        if (r & 1) ps1 += pv; else ps0 += pv;
        pop[st][r >> 3][r & 7] = (__bf16)pv;
      }
    float psum = ps0 + ps1;
    if (__ballot(!(psum <= kMaxWeightSum))) {
      __asm__ volatile("" ::);
      float mx = s[0][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[0][r]);
#pragma unroll
      for (int st = 1; st < NST; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[st][r]);
      mx = xor32_max(mx);
      const bool grow = mx * c > m_run + kMaxLag;
      const float m_new = grow ? mx * c : m_run;
      const float alpha = grow ? fexp2(m_run - m_new) : 1.0f;
      ps0 = ps1 = 0.f;
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float pv = fexp2(__builtin_fmaf(s[st][r], c, -m_new));
          if (r & 1) ps1 += pv; else ps0 += pv;
          pop[st][r >> 3][r & 7] = (__bf16)pv;
        }
      psum = ps0 + ps1;
      l_run *= alpha;
      if (__ballot(grow)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[mb][r] *= alpha;
      }
      m_run = m_new;
    }
    l_run += psum;
  };
  // end of phase t: at t = 2i, wait for this wave's copies of V(i) and everything before it (K(i + 1)
  // among them), which M(i + 1) reads from phase 2i + 2 on and the softmax phase before it reads
  // ahead (the copy of K(i + 2), issued since, stays in flight); then drain the LDS reads and pass
  // the barrier without the release fence of __syncthreads (which would drain every copy)
  constexpr int P = DT::NDMA;                       // DMA instructions per tensor and stage
  auto end_phase = [&](int t) {
    if ((t & 1) == 0) {
      const int i = t >> 1;
      if (i + 2 < n) __builtin_amdgcn_s_waitcnt(PEARL_VMCNT(P));   // K(i + 2) stays in flight
      else __builtin_amdgcn_s_waitcnt(PEARL_VMCNT(0));
    }
    __builtin_amdgcn_s_waitcnt(PEARL_LGKMCNT0);
    __asm__ volatile("s_barrier" ::: "memory");
  };

  // prologue: K(0), V(0), K(1), and zeros into V buffer 2 (read by M(0), whose P is 0; V(2) is
  // copied there only with the pair 1); the first M phase needs K(0).  Block-table entries are
  // read in softmax phases, a phase or more before they are used: scalar loads share the LDS
  // reads' counter and complete out of order, so one in flight during an M phase would make
  // every operand wait drain the counter, and one used right away would stall the phase for a
  // memory round trip.  The end-of-phase drain completes them.
  {
    const int p0 = page_of(0);
    dma(0, false, p0, kbuf(0));
    dma(0, true, p0, vbuf(0));
  }
  if (1 < n) dma(1, false, pid_v, kbuf(1));
#pragma unroll
  for (int i = 0; i < DT::NDMA; ++i)
    lds_dma16_untracked(zero_src, vbuf(2) + (DT::RPW * w + DT::RPI * i) * RB);
  __builtin_amdgcn_s_waitcnt(PEARL_VMCNT(0));       // Q loads and the first copies (also this item's)
  __asm__ volatile("s_barrier" ::: "memory");
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  // Each group runs its own loop (the same barriers in the same number: 2n + 2), so the registers
  // of S and P are never live together on any path.  The loops are unrolled over the three buffers
  // and no phase is conditional inside them.
  if (grp == 0) {
    // phases 2j, 2j + 1 for j < n: M(j), V(j); then M(n) and an empty phase.  The K rows of the
    // pair follow the MFMAs of M(j), the V rows open V(j), and the block-table entry of the next K
    // rows is read during V(j).
    auto step = [&](auto r_c, int j, auto first_c) {
      constexpr int R = decltype(r_c)::value;
      phase_m(r_c, !decltype(first_c)::value);
      copy_k(r_c, j);
      end_phase(2 * j);
      copy_v(r_c, j);
      pid_v = pid_k;
      if (j + 3 < n) pid_k = page_of(j + 3);
      phase_v(j);
      prefetch(std::integral_constant<int, (R + 1) % 3>{});
      end_phase(2 * j + 1);
    };
    using F = std::false_type;
    step(I0{}, 0, std::true_type{});                // n >= 1
    int j = 1;
    for (; j + 3 <= n; j += 3) {
      step(I1{}, j, F{});
      step(I2{}, j + 1, F{});
      step(I0{}, j + 2, F{});
    }
    if (j < n) { step(I1{}, j, F{}); ++j; }
    if (j < n) { step(I2{}, j, F{}); ++j; }
    const int r = n % 3;                            // j == n
    if (r == 0) phase_m(I0{}, true); else if (r == 1) phase_m(I1{}, true); else phase_m(I2{}, true);
    end_phase(2 * n);
    end_phase(2 * n + 1);
  } else {
    // phases 0, 1: an empty phase, M(0); phases 2j, 2j + 1 for 1 <= j <= n: V(j - 1), M(j).  The
    // K rows of pair j open V(j - 1) (phase 0 for pair 0), the V rows follow the MFMAs of M(j),
    // and the block-table entry of the K rows after them is read during V(j - 1).
    auto pair_done = [&]() {
      pid_v = pid_k;
      pid_k = pid_n;
    };
    auto step = [&](auto r_c, int j) {
      copy_k(r_c, j);
      if (j + 3 < n) pid_n = page_of(j + 3);
      phase_v(j - 1);
      prefetch(r_c);
      end_phase(2 * j);
      phase_m(r_c, true);
      copy_v(r_c, j);
      pair_done();
      end_phase(2 * j + 1);
    };
    copy_k(I0{}, 0);
    if (3 < n) pid_n = page_of(3);
    end_phase(0);
    phase_m(I0{}, false);
    copy_v(I0{}, 0);
    pair_done();
    end_phase(1);
    int j = 1;
    for (; j + 3 <= n + 1; j += 3) {
      step(I1{}, j);
      step(I2{}, j + 1);
      step(I0{}, j + 2);
    }
    if (j <= n) { step(I1{}, j); ++j; }
    if (j <= n) { step(I2{}, j); ++j; }
  }


  at_end();
  // epilogue: combine the two half-row sums; a split item stores its fp32 partial state, a whole
  // item normalises and stores bf16 O and the fp32 LSE
  const float l_tot = xor32_add(l_run);
  if (row_ok && n_split > 1) {
    const int slot = a.split_base[b] + split * ((si.q_len + a.tokens_per_tile - 1) / a.tokens_per_tile) + tile;
    const size_t prow = (size_t)(slot * H_kv + g) * kRowsPerTile + rho;
    float* po = a.part_pre_o + prow * D;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        *reinterpret_cast<f32x4*>(po + 32 * mb + 8 * rq + 4 * half) =
            f32x4{oacc[mb][4 * rq + 0], oacc[mb][4 * rq + 1], oacc[mb][4 * rq + 2], oacc[mb][4 * rq + 3]};
    if (half == 0) {
      a.part_pre_ml[2 * prow] = m_run;
      a.part_pre_ml[2 * prow + 1] = l_tot;
    }
  } else if (row_ok) {
    const float inv = 1.0f / l_tot;
    uint16_t* orow = a.out + ((size_t)(si.q_start + tok) * H_q + h) * D;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int dim = 32 * mb + 8 * rq + 4 * half;
        u32x2 pk;
        pk[0] = (uint32_t)bf16_bits(oacc[mb][4 * rq + 0] * inv) | ((uint32_t)bf16_bits(oacc[mb][4 * rq + 1] * inv) << 16);
        pk[1] = (uint32_t)bf16_bits(oacc[mb][4 * rq + 2] * inv) | ((uint32_t)bf16_bits(oacc[mb][4 * rq + 3] * inv) << 16);
        *reinterpret_cast<u32x2*>(orow + dim) = pk;
      }
    if (half == 0 && a.lse) a.lse[(size_t)(si.q_start + tok) * H_q + h] = (m_run + flog2(l_tot)) * kLn2;
  }
}

// ------------------------------------------------------------------------------------------------
// Decode work item: one (sequence, kv-head g, split of pps pages; the planner chooses pps).  The
// G q-heads of the group are the 16 columns of the MFMA products (columns >= G are zero), so each
// K/V byte is loaded once for the whole group.  Wave w takes pages w, w+8, ... of the split:
//   S^T (16 keys x heads) = K_page . Q^T           (16x16x32 MFMA: A = K rows read from LDS)
//   O^T (dims x heads)   += V^T . P^T over 16 keys (16x16x16 MFMA: A = V^T read transposed from LDS)
// K and V travel HBM -> LDS by 16-byte LDS-DMA loads (no VGPRs, no LDS store instructions) into a
// per-wave double buffer, so the next page's loads are in flight while the current page is
// consumed.  Each DMA instruction moves whole key rows (1 KiB of consecutive bytes), marked
// non-temporal: every K/V byte is read once per launch, and such full-line reads marked that way
// reach a higher HBM rate than plain ones (K read straight into MFMA operand registers touched
// half of each 128-byte line per instruction, which the non-temporal mark made slower).  Every
// load is unconditional: addresses stay inside the split's own pages, and V rows of keys past the
// sequence end are fetched from a zeroed block of the workspace so they add nothing to P.V
// (their scores are masked to -inf).  The 8 waves' partial softmax states are merged through
// LDS; a sequence with one split writes its output directly, otherwise the (o~, m, l) partial
// goes to the workspace.
//
// Stage layout (per wave): the page's K rows, then its V rows, kPage rows x D/8 16-byte chunks
// each, unpadded.  Chunk c of K row r sits in slot c ^ kswz(r), so the 16 rows that one operand
// read covers fall in 16 different 16-byte bank groups; chunk c of V row r sits in slot
// c ^ vswz(r), which spreads the transposing reads over all LDS banks.
// ------------------------------------------------------------------------------------------------
template <int D> struct PageTile {
  static constexpr int CPR = D / 8;                 // 16-byte chunks per key row
  static constexpr int ROWB = D * 2;                // bytes per key row
  static constexpr int RPI = 64 / CPR;              // rows written by one 64-lane DMA instruction
  static constexpr int TBYTES = kPage * ROWB;       // one tensor of one page
  static constexpr int BYTES = 2 * TBYTES;          // K rows, then V rows
  static constexpr int NDMA = kPage / RPI;          // DMA instructions per tensor and page
  static constexpr int KB = D / 32;                 // 32-wide k blocks of the QK product
  static constexpr int MB = D / 16;                 // 16-wide dim blocks of the PV product
  __device__ static __forceinline__ int kswz(int r) {
    // d = 128: 16 slots per row, one per row of the page; d = 64: 8 slots per row and rows 2i,
    // 2i + 1 in opposite halves of the banks
    if constexpr (D == 128) return r & 15;
    else return (r >> 1) & 7;
  }
  __device__ static __forceinline__ int vswz(int r) {
    return (((r & 3) << 2) | (((r >> 2) & 1) << 1)) & (CPR - 1);
  }
  // byte offset of K row r, chunk c
  __device__ static __forceinline__ int koff(int r, int c) { return r * ROWB + ((c ^ kswz(r)) << 4); }
  // byte offset of (V row r, 4-element group starting at dim d0)
  __device__ static __forceinline__ int voff(int r, int d0) {
    return TBYTES + r * ROWB + (((d0 >> 3) ^ vswz(r)) << 4) + ((d0 >> 2) & 1) * 8;
  }
};


// The new token's K/V row of a fused append-and-decode: logical page `page`, slot `slot`, taken
// from the caller's k_new / v_new rows instead of the pool (page -1: none).
struct NewRow {
  int page, slot;
  const uint16_t* k;
  const uint16_t* v;
};

// Issues the copies of logical page p (physical page phys) of kv-head g into the stage at dst.
// kNew: the item may hold the new row (decode_kernel); otherwise nr is ignored.
template <int D, bool kNew>
__device__ __forceinline__ void decode_issue(const AttnArgs& a, int phys, int p, int g, int kv, char* dst,
                                             const NewRow& nr) {
  using PT = PageTile<D>;
  const int lane = threadIdx.x & 63;
  const size_t blk = ((size_t)phys * a.num_kv_heads + g) * (size_t)(kPage * D);
  const uint16_t* zero = reinterpret_cast<const uint16_t*>(a.ws_hdr + kHdrZero);
  const int slot = lane % PT::CPR;                  // chunk slot this lane fills
#pragma unroll
  for (int i = 0; i < PT::NDMA; ++i) {
    const int r = i * PT::RPI + lane / PT::CPR;     // key row of the page written by this lane
    const bool is_new = kNew && p == nr.page && r == nr.slot;
    const int ck = slot ^ PT::kswz(r);
    lds_dma16_untracked<true>(is_new ? nr.k + ck * 8 : a.k_pool + blk + r * D + ck * 8, dst + i * 1024);
  }
#pragma unroll
  for (int i = 0; i < PT::NDMA; ++i) {
    const int r = i * PT::RPI + lane / PT::CPR;
    const bool ok = p * kPage + r < kv;
    const bool is_new = kNew && p == nr.page && r == nr.slot;
    const int cv = slot ^ PT::vswz(r);
    const uint16_t* src = ok ? (is_new ? nr.v + cv * 8 : a.v_pool + blk + r * D + cv * 8) : zero;
    lds_dma16_untracked<true>(src, dst + PT::TBYTES + i * 1024);
  }
}

// The copies of a whole page (the stage layout of decode_issue): the lanes' byte offsets in a block
// are the same for every page, so a page costs its two block addresses and the copies themselves.
// An instruction's immediate offset advances the source and the LDS address alike.
template <int D> struct PageCopies {
  using PT = PageTile<D>;
  int k[PT::NDMA], v[PT::NDMA];
  __device__ __forceinline__ explicit PageCopies(int lane) {
    const int slot = lane % PT::CPR, r0 = lane / PT::CPR;
#pragma unroll
    for (int i = 0; i < PT::NDMA; ++i) {            // less the immediate offset, i 1024
      const int r = i * PT::RPI + r0;
      k[i] = r0 * PT::ROWB + ((slot ^ PT::kswz(r)) << 4);
      v[i] = r0 * PT::ROWB + ((slot ^ PT::vswz(r)) << 4);
    }
  }
  // kb, vb: the blocks (uniform); dst: the stage (uniform)
  __device__ __forceinline__ void issue(const uint16_t* kb, const uint16_t* vb, const char* dst) const {
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)((LDS_AS const char*)dst));
    unsigned saved;
    if constexpr (D == 128) {
      static_assert(PT::NDMA == (D == 128 ? 4 : 2) && PT::TBYTES == PT::NDMA * 1024, "page copies");
      __asm__ volatile(
          "s_mov_b32 %0, m0\n\t"
          "s_mov_b32 m0, %1\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %4, %2 nt\n\t"
          "global_load_lds_dwordx4 %5, %2 offset:1024 nt\n\t"
          "global_load_lds_dwordx4 %6, %2 offset:2048 nt\n\t"
          "global_load_lds_dwordx4 %7, %2 offset:3072 nt\n\t"
          "s_add_u32 m0, %1, 0x1000\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %8, %3 nt\n\t"
          "global_load_lds_dwordx4 %9, %3 offset:1024 nt\n\t"
          "global_load_lds_dwordx4 %10, %3 offset:2048 nt\n\t"
          "global_load_lds_dwordx4 %11, %3 offset:3072 nt\n\t"
          "s_mov_b32 m0, %0"
          : "=&s"(saved)
          : "s"(lds), "s"(kb), "s"(vb), "v"(k[0]), "v"(k[1]), "v"(k[2]), "v"(k[3]), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3])
          : "memory", "scc");
    } else {
      __asm__ volatile(
          "s_mov_b32 %0, m0\n\t"
          "s_mov_b32 m0, %1\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %4, %2 nt\n\t"
          "global_load_lds_dwordx4 %5, %2 offset:1024 nt\n\t"
          "s_add_u32 m0, %1, 0x800\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %6, %3 nt\n\t"
          "global_load_lds_dwordx4 %7, %3 offset:1024 nt\n\t"
          "s_mov_b32 m0, %0"
          : "=&s"(saved)
          : "s"(lds), "s"(kb), "s"(vb), "v"(k[0]), "v"(k[1]), "v"(v[0]), "v"(v[1])
          : "memory", "scc");
    }
  }
};

// A page's copies: whole pages by PageCopies, the sequence's last one with its rows past the end.
template <int D>
__device__ __forceinline__ void issue_whole_or_last(const AttnArgs& a, int phys, int p, int g, int kv, char* dst,
                                                    const PageCopies<D>& copies) {
  if ((p + 1) * kPage <= kv) {
    const size_t blk = ((size_t)phys * a.num_kv_heads + g) * (size_t)(kPage * D);
    copies.issue(a.k_pool + blk, a.v_pool + blk, dst);
  } else {
    decode_issue<D, false>(a, phys, p, g, kv, dst, NewRow{-1, 0, nullptr, nullptr});
  }
}

// Attends the G heads to logical page p staged at buf, updating the wave's online softmax state.
// kFine: the weights enter P.V as two bf16 parts, the upper 8 significant bits (cut off, so the rest
// is >= 0) and the rest, in a product each on the same V operand (side by side in one 16x16x32
// product the operand had to be copied, which cost calls 0.1-0.4 us).
// Rounded to bf16 once, a weight is off by up to 2^-9 unless it is the largest of its run, which is
// exactly 1: the fewer runs a sequence is cut into, the larger the error, and the equal shares'
// long runs took the error of 64 sequences of 2K-16K tokens from 0.00177 to 0.00185 (2-norm, against
// 64 bits); in two parts it is 0.00166, that of rounding the exact result to bf16.
template <int D, bool kFine>
__device__ __forceinline__ void decode_consume(int p, int kv, const bf16x8* qop, f32x4* oacc, float& m_run,
                                               float& l_run, const float c, const char* buf) {
  using PT = PageTile<D>;
  const int lane = threadIdx.x & 63, gi = lane >> 4, j = lane & 15;
  // S^T: lane l holds head l % 16 of keys 4 gi .. 4 gi + 3; its K operand is row l % 16, dims of
  // chunk 4 kb + gi (the Q operand holds the same dims)
  f32x4 sc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < PT::KB; ++kb) {
    const bf16x8 kop = *reinterpret_cast<const bf16x8*>(buf + PT::koff(j, 4 * kb + gi));
    sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop, qop[kb], sc, 0, 0, 0);
  }
  // mask keys past the end of the sequence (a select, so stray bit patterns never leak)
#pragma unroll
  for (int r = 0; r < 4; ++r) sc[r] = (p * kPage + 4 * gi + r < kv) ? sc[r] : -INFINITY;
  float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  // the maximum only moves when this page exceeds it, and the O rescale is skipped when no lane
  // of the wave moved (decode is bound by HBM, so it keeps the exact maximum)
  const bool grow = mx * c > m_run;
  const float m_new = grow ? mx * c : m_run;
  const float alpha = grow ? fexp2(m_run - m_new) : 1.0f;
  i16x4 pop, rest;
  float psum = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float pr = fexp2(__builtin_fmaf(sc[r], c, -m_new));
    psum += pr;
    if constexpr (kFine) {
      const unsigned upper = __builtin_bit_cast(unsigned, pr) & 0xffff0000u;
      pop[r] = (short)(upper >> 16);
      // never 0 unless the weight is, so an infinite V stays infinite (0 times it would be NaN)
      rest[r] = (short)bf16_bits(fmaxf(pr - __builtin_bit_cast(float, upper), fminf(pr, 0x1p-100f)));
    } else {
      pop[r] = (short)bf16_bits(pr);
    }
  }
  l_run = l_run * alpha + psum;
  if (__ballot(grow)) {
#pragma unroll
    for (int mb = 0; mb < PT::MB; ++mb) oacc[mb] *= alpha;
  }
  m_run = m_new;
  // O^T += V^T P^T: the transposing read gives lane l dim 16 mb + l % 16 of keys 4 gi .. 4 gi + 3,
  // the k index of the P^T operand that lane already holds
  const int r0 = 4 * gi + (j >> 2);
  i16x4 v[PT::MB];
#pragma unroll
  for (int mb = 0; mb < PT::MB; ++mb) {
    v[mb] = lds_read_tr(buf, PT::voff(r0, 16 * mb + 4 * (j & 3)));
    oacc[mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[mb], pop, oacc[mb], 0, 0, 0);
  }
  if constexpr (kFine) {
#pragma unroll
    for (int mb = 0; mb < PT::MB; ++mb) oacc[mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v[mb], rest, oacc[mb], 0, 0, 0);
  }
}


// Physical page of logical page p of the row, read with a scalar load from the block table.
__device__ __forceinline__ int page_id(ConstI32Ptr bt_row, int p, int num_pages) {
  return clamp_page(bt_row[p], num_pages);
}

// One decode work item as the kernels see it: sequence b (its new token is row q_row of q/out),
// kv attended keys, split `split` of n_splits (pps pages each), kv-head g; the partials of a
// multi-split sequence go to slots slot_base + split.
struct DecItem {
  int b, split, g, q_row, kv, n_splits, slot_base;
};

// One pipeline step: issue the next page's copies into s_next (when the wave has one: `more`,
// wave-uniform), then wait for the current page's and consume it from s_cur.  The copies are
// issued untracked, so the compiler adds no waits of its own for them (left to itself it drained
// every copy in flight in one of the loop's two unrolled steps); s_next was last read in the
// previous step, whose operand reads all completed before its MFMAs.
template <int D>
__device__ __forceinline__ void decode_step(const AttnArgs& a, int p_cur, int p_nxt, int phys_nxt, int g, int kv,
                                            char* __restrict__ s_next, const char* __restrict__ s_cur,
                                            const bf16x8* qop, f32x4* oacc, float& m_run, float& l_run,
                                            const PageCopies<D>& copies, bool more) {
  constexpr int PAGE_LOADS = 2 * PageTile<D>::NDMA;   // vector-memory ops per page
  // the current page has landed; the copies are invisible to the compiler, so the wait is also a
  // compiler barrier that keeps the stage reads below it
  if (more) {
    issue_whole_or_last<D>(a, phys_nxt, p_nxt, g, kv, s_next, copies);
    __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"(PAGE_LOADS) : "memory");
  } else {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  decode_consume<D, false>(p_cur, kv, qop, oacc, m_run, l_run, a.scale_log2, s_cur);
}

// One decode item of a launch planned by plan_kernel; its partials are merged by merge_kernel after
// the launch.
template <int D, int NW, typename AtEnd>
__device__ __forceinline__ void decode_split(const AttnArgs& a, const DecItem& it, int pps, char* stageA,
                                             char* stageB, AtEnd at_end) {
  constexpr int NT = NW * 64;
  using PT = PageTile<D>;
  constexpr int MB = PT::MB;
  constexpr int KB = PT::KB;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index (uniform)
  const int gi = lane >> 4, hh = lane & 15;
  const int b = it.b, split = it.split, g = it.g;
  const int G = a.group, H_q = a.num_q_heads;
  const int kv = it.kv;
  const int n_pages = (kv + kPage - 1) / kPage;
  const int p_begin = split * pps;
  const int p_end = min(p_begin + pps, n_pages);
  const int n_pg = p_end - p_begin;                 // pages of this split (>= 1)
  const bool head_ok = hh < G;
  char* st0 = stageA + w * PT::BYTES;
  char* st1 = stageB + w * PT::BYTES;

  const ConstI32Ptr bt_row = (ConstI32Ptr)(a.block_table + (size_t)b * a.bt_stride);

  bf16x8 qop[KB];
  {
    const uint16_t* qrow = a.q + ((size_t)it.q_row * H_q + g * G + (head_ok ? hh : 0)) * D + 8 * gi;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const bf16x8 v = as_bf16x8(ld16(qrow + 32 * kb));
      qop[kb] = head_ok ? v : zero_bf16x8();
    }
  }
  // the page ids run one page ahead of the copies, which run one page ahead of the compute
  int cur = min(w, n_pg - 1);
  int ph_cur = page_id(bt_row, p_begin + cur, a.num_pages);
  const PageCopies<D> copies(lane);
  if (w < n_pg) issue_whole_or_last<D>(a, ph_cur, p_begin + cur, g, kv, st0, copies);
  f32x4 oacc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) oacc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;

  // page indices past the wave's last page are clamped to the split's last page; such a page id is
  // read but never copied
  int nxt = min(w + NW, n_pg - 1);
  int ph_nxt = page_id(bt_row, p_begin + nxt, a.num_pages);
  for (int pi = w; pi < n_pg; pi += 2 * NW) {
    const int pj = pi + NW;
    const int n2 = min(pj + NW, n_pg - 1);
    const int ph_n2 = page_id(bt_row, p_begin + n2, a.num_pages);
    decode_step<D>(a, p_begin + cur, p_begin + nxt, ph_nxt, g, kv, st1, st0, qop, oacc, m_run, l_run, copies, pj < n_pg);
    if (pj >= n_pg) break;
    const int n3 = min(pj + 2 * NW, n_pg - 1);
    const int ph_n3 = page_id(bt_row, p_begin + n3, a.num_pages);
    decode_step<D>(a, p_begin + nxt, p_begin + n2, ph_n2, g, kv, st0, st1, qop, oacc, m_run, l_run, copies,
                   pj + NW < n_pg);
    cur = n2;
    nxt = n3;
    ph_nxt = ph_n3;
  }
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // each head's four lane groups hold different keys: sum their l
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);

  at_end();
  // merge the waves' states through LDS
  __syncthreads();
  static_assert(Lds<D, NW, 2>::merge_bytes <= NW * PT::BYTES, "merge scratch fits in one set of stages");
  float* mo = reinterpret_cast<float*>(stageA);               // [wave][8 heads][D]
  float* mm = mo + NW * 8 * D;                            // [wave][8]
  float* ml = mm + NW * 8;                                // [wave][8]
  if (head_ok) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      *reinterpret_cast<f32x4*>(mo + (w * 8 + hh) * D + 16 * mb + 4 * gi) = oacc[mb];
    if (gi == 0) { mm[w * 8 + hh] = m_run; ml[w * 8 + hh] = l_run; }
  }
  __syncthreads();
  const int n_splits = it.n_splits;
  for (int t = threadIdx.x; t < G * D; t += NT) {
    const int head = t / D, dim = t - head * D;
    float M = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) M = fmaxf(M, mm[ww * 8 + head]);
    float L = 0.f, o = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const float f = fexp2(mm[ww * 8 + head] - M);
      L += f * ml[ww * 8 + head];
      o += f * mo[(ww * 8 + head) * D + dim];
    }
    const int hq = g * G + head;
    if (n_splits == 1) {
      a.out[((size_t)it.q_row * H_q + hq) * D + dim] = bf16_bits(o / L);
      if (dim == 0 && a.lse) a.lse[(size_t)it.q_row * H_q + hq] = (M + flog2(L)) * kLn2;
    } else {
      const size_t pidx = (size_t)(it.slot_base + split) * H_q + hq;
      a.part_o[pidx * D + dim] = o;
      if (dim == 0) { a.part_ml[2 * pidx] = M; a.part_ml[2 * pidx + 1] = L; }
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// Persistent attention kernel: workgroups take items (entry x kv-head) from the planner's list
// through atomic counters (the next item is claimed as the current one ends); prefill tiles
// come first (largest work), decode splits fill the tail.
// ------------------------------------------------------------------------------------------------
// kKinds: 1 = prefill tiles only, 2 = decode splits only, 3 = both (mixed batches).
template <int D, int kKinds> struct KernelCfg {
  static constexpr int NW = kWaves;
  static constexpr int NT = NW * 64;
};

template <int D, int kKinds>
__global__ __launch_bounds__((KernelCfg<D, kKinds>::NT)) void attn_kernel(AttnArgs a, int max_pre) {
  constexpr int NW = KernelCfg<D, kKinds>::NW;
  __shared__ __attribute__((aligned(16))) char smem[Lds<D, NW, kKinds>::bytes];
  // the two stages of the decode pipeline are separate objects so the LDS reads of one are
  // known not to alias the LDS-DMA writes still in flight into the other
  __shared__ __attribute__((aligned(16))) char stageA_[(kKinds == 2) ? NW * PageTile<D>::BYTES : 16];
  __shared__ __attribute__((aligned(16))) char stageB_[(kKinds == 2) ? NW * PageTile<D>::BYTES : 16];
  char* stageA = (kKinds == 2) ? stageA_ : smem;
  char* stageB = (kKinds == 2) ? stageB_ : smem + NW * PageTile<D>::BYTES;
  // prefill-only kernels: three K and three V stage buffers, each set contiguous
  constexpr int kDT = (kKinds == 1) ? DmaTile<D>::BYTES : 16;
  __shared__ __attribute__((aligned(16))) char pk[3 * kDT], pv[3 * kDT];
  __shared__ int s_item[2][2];                      // next item and claim mode
  const int n_items = a.ws_hdr[kHdrNumItems];
  const int n_pre = a.ws_hdr[kHdrNumPre];
  const int pps = a.ws_hdr[kHdrPagesPerSplit];
  const int H_kv = a.num_kv_heads;
  // Items: prefill items [0, n_pre * H_kv), decode items after them.  Every workgroup's first item
  // follows from its index: workgroups below pre_wgs (all in prefill launches, the planner's
  // kHdrPreFirstWG in mixed ones) start with prefill items and keep to them while there are any, the
  // others with decode items, so both kinds run side by side; each takes the other kind once its
  // own is exhausted.  The following items are claimed at the end of the one before: claimed a whole
  // item ahead, the longest-first order loses its balance (348 items on 256 units wait for the
  // second of two that one unit holds: 46 stages against 34).  The claim goes out before the item's
  // epilogue, which hides most of its latency.
  // Before, every workgroup's first claim waited for 256 others on the counters, and at its end it
  // asked all 8 queues one after the other while its last item waited for the answer: 28 chunks of
  // 26 tokens on 40-80 cached ones took 47 us a call and take 24 (kernel 39 -> 17), one prompt of
  // 2000 tokens 87 -> 72, 24 decodes beside a 256-token chunk 140 -> 129.
  const int n_pre_items = n_pre * H_kv, n_dec_items = n_items - n_pre_items;
  const int grid = gridDim.x;
  const int pre_wgs = kKinds == 1 ? grid : kKinds == 2 ? 0 : min(a.ws_hdr[kHdrPreFirstWG], grid);
  const int dec_wgs = grid - pre_wgs;
  const bool pre_first = (int)blockIdx.x < pre_wgs;
  // Prefill items: item i belongs to queue i % 8, and a workgroup takes the items of the queue of
  // the XCD it runs on, then those of the other queues in turn.  With 8 kv-heads the items of
  // one (sequence, kv-head) then share one XCD's L2 (with 4, two XCDs): every tile of a sequence
  // re-reads that head's whole context, which other XCDs would each fetch from memory again.  The
  // queues are balanced (the heads of a tile are equal work), and the turn to other queues
  // completes every item wherever the workgroups run.  Claim c of queue q is its item after those
  // the workgroups started with.
  auto pre_item = [&](int q, int c) { return (unsigned)q + kNumXcd * (unsigned)(c + ((pre_wgs - q + kNumXcd - 1) >> 3)); };
  static_assert(kNumXcd == 8, "queue arithmetic");
  const int xcd = xcc_id();
  // What the next claim tries: 0 nothing (every item is some workgroup's first one), 1 this XCD's
  // prefill queue, 2 the decode counter.
  const bool any_pre = (kKinds & 1) && n_pre_items > pre_wgs, any_dec = (kKinds & 2) && n_dec_items > dec_wgs;
  int mode = pre_first ? (any_pre ? 1 : any_dec ? 2 : 0) : (any_dec ? 2 : any_pre ? 1 : 0);
  int claimed = 0;                                  // thread 0's
  auto send_claim = [&]() {
    if (mode != 0 && threadIdx.x == 0) claimed = atomicAdd(&a.ws_hdr[mode == 1 ? kHdrQueues + xcd : kHdrCounter], 1);
  };
  // Wave 0, after send_claim: the next item (-1: none left) to s_item[slot], the next mode beside it.
  // If the tried kind is exhausted here, one read of all queue counters finds a queue that still
  // holds items, so an exhausted launch costs one round trip and not one per queue.
  auto take_claim = [&](int slot) {
    const int c = __builtin_amdgcn_readfirstlane(claimed), lane = threadIdx.x;
    int next = -1, next_mode = mode;
    if (mode == 1) {
      if (pre_item(xcd, c) < (unsigned)n_pre_items) next = (int)pre_item(xcd, c);
    } else if (dec_wgs + c < n_dec_items) {
      next = n_pre_items + dec_wgs + c;
    }
    for (int tries = 0; tries < 2 && next < 0; ++tries) {   // the other queues, or the other kind
      if (any_pre && (mode == 1) == (tries == 0)) {
        for (;;) {
          const int n = __hip_atomic_load(&a.ws_hdr[kHdrQueues + (lane & 7)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const unsigned has = (unsigned)__ballot(lane < kNumXcd && pre_item(lane, n) < (unsigned)n_pre_items);
          if (!has) break;
          const int q = (xcd + __builtin_ctz((has >> xcd) | (has << (kNumXcd - xcd)))) & 7;   // own queue first
          int got = 0;
          if (lane == 0) got = atomicAdd(&a.ws_hdr[kHdrQueues + q], 1);
          const unsigned i = pre_item(q, __builtin_amdgcn_readfirstlane(got));
          if (i < (unsigned)n_pre_items) { next = (int)i; next_mode = 1; break; }   // else taken meanwhile
        }
      } else if (any_dec && mode == 1) {
        int got = 0;
        if (lane == 0) got = atomicAdd(&a.ws_hdr[kHdrCounter], 1);
        got = dec_wgs + __builtin_amdgcn_readfirstlane(got);
        if (got < n_dec_items) { next = n_pre_items + got; next_mode = 2; }
      }
    }
    if (lane == 0) { s_item[slot][0] = next; s_item[slot][1] = next_mode; }
  };
  int item = pre_first ? ((int)blockIdx.x < n_pre_items ? (int)blockIdx.x : -1)
                       : ((int)blockIdx.x - pre_wgs < n_dec_items ? n_pre_items + (int)blockIdx.x - pre_wgs : -1);
  int slot = 0;
  auto go_on = [&]() {                              // after send_claim, by all threads
    if (threadIdx.x < 64) take_claim(slot);
    __syncthreads();
    item = __builtin_amdgcn_readfirstlane(s_item[slot][0]);
    mode = __builtin_amdgcn_readfirstlane(s_item[slot][1]);
    slot ^= 1;
  };
  if (item < 0 && mode != 0) {                      // none of the own kind to start with
    send_claim();
    go_on();
  }
  while (item >= 0) {
    const int e = item / H_kv;
    const int g = item - e * H_kv;
    if (e < n_pre) {
      if constexpr ((kKinds & 1) != 0) {
        static_assert(NW == kWaves, "prefill tiles use 8 waves");
        const int2 en = a.entries[e];
        if constexpr (kKinds == 1) {
          prefill_tile_pp<D>(a, en.x, en.y, g, pk, pv, send_claim);
        } else {
          // the mixed kernel's prefill stage buffers share its LDS region with the decode stages (a
          // workgroup runs one item at a time, and items are separated by a drained barrier)
          constexpr int B = DmaTile<D>::BYTES;
          static_assert(6 * B <= Lds<D, NW, kKinds>::bytes, "stage buffers fit the shared region");
          prefill_tile_pp<D>(a, en.x, en.y, g, smem, smem + 3 * B, send_claim);
        }
      }
    } else {
      if constexpr ((kKinds & 2) != 0) {
        const int2 en = a.entries[max_pre + (e - n_pre)];
        const SeqInfo si = a.seqinfo[en.x];
        const DecItem it{en.x, en.y, g, si.q_start, si.ctx_len + si.q_len, si.kind >> 4, a.split_base[en.x]};
        decode_split<D, NW>(a, it, pps, stageA, stageB, send_claim);
      }
    }
    if (mode == 0) break;
    go_on();
  }
}

// ------------------------------------------------------------------------------------------------
// Decode of batches of up to kDecPlanMaxSeqs sequences: one launch of equal shares.
//
// The work of one kv-head is the list of the batch's pages in (sequence, page) order.  The list is
// cut into equal shares, one per wave, so every wave streams the same number of pages whatever
// the lengths are, and its double buffer of page copies never drains between the sequences it
// passes through.  A workgroup holds consecutive shares of one kv-head, or the same shares of up
// to 8 kv-heads (DecShares).
//   * A (sequence, kv-head) pair inside one share is normalised and stored by its wave alone.
//   * A pair cut by share boundaries leaves a partial (o~, m, l) in each wave: at most two per wave,
//     the first pair's (kept in registers until the share ends) and the last one's.  At the end
//     the workgroup merges those of each kv-head through LDS.
//   * A pair cut by workgroup boundaries leaves at most two partials per workgroup and kv-head in
//     the workspace (a first slot for the pair holding its first page, a second one for another
//     pair), merged by the workgroup that finishes last.
// What bounds it: the HBM read rate while it streams (decode-64 below reads 6.9 TB/s from the first
// page to the last wave's end, the rate of a plain non-temporal read), then about 10 us of latency
// a launch: lengths, page id and first page one after the other (3-4 us), the LDS merge, the
// store acknowledgement, the count-in and the last merge (5-8 us).  Before, splits of equal size
// came from a work queue and each drained its pipeline and merged 8 waves (3.6 us per split, and a
// tail of a split's length).  Times of a call, before and now (32 q-heads, d = 128 unless said;
// same card, in turn): 64 sequences of 2K-16K tokens, 8 kv-heads 362 -> 352 us; 256 around 6K
// tokens, 4 kv-heads 647 -> 632 (both 2-4% over batches of other such lengths); 512 of 64-1024 tokens
// 202 -> 190; 32 around 6K, 4 kv-heads 93.4 -> 82.8; 48 of 500-6000 tokens, 16 q-heads, 8 kv-heads,
// d = 64 60.8 -> 55.5; one of 2731 tokens 14.6 -> 13.2, of 16000 34.0 -> 21.4; 200 of 40-160 tokens
// 37.5 -> 24.8.
// The shares follow from the lengths alone, so results do not depend on timing.  Every workgroup
// finds its place by itself from the prefix sums of the pages per sequence (decode_plan), so the
// call is a zeroing launch and this kernel.
// ------------------------------------------------------------------------------------------------
constexpr int kDecPlanChunks = kDecPlanMaxSeqs / kThreads;
static_assert(kDecPlanChunks * kThreads == kDecPlanMaxSeqs, "plan chunks");

struct DecPlanLds {
  int pre[kDecPlanMaxSeqs + 1];            // exclusive prefix sums of pages
  unsigned char tail[kDecPlanMaxSeqs];     // (attended keys - 1) % kPage
  int wsum[kWaves];
  int err;
  int over;                                // a sequence is longer than all_within's limit
};

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Pages and attended keys of one sequence from its length; false if it violates the host bounds.
__device__ __forceinline__ bool dec_seq(const AttnArgs& a, const DecPlanArgs& d, int b, int& pages, int& tail) {
  const int ctx = d.ctx_lens[b];
  const long long kv = (long long)ctx + 1;
  if (ctx < 0 || kv > d.max_kv_len || (kv + kPage - 1) / kPage > a.bt_stride) return false;
  pages = (int)((kv + kPage - 1) / kPage);
  tail = ctx % kPage;
  return true;
}

// Builds the prefix sums; returns the total pages, or -1 if a length violates the host bounds.
// most: the most pages of this thread's sequences (of this lane's: every wave holds them all).
// Batches of at most 64 sequences: every wave builds the same list (the same values to the same
// words), a lane per sequence, so no barrier is needed; a wave reads other lanes' words only after
// the fence that orders its own stores before them.
__device__ __forceinline__ int decode_plan(const AttnArgs& a, const DecPlanArgs& d, DecPlanLds& P, int& most) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, B = d.batch;
  // inclusive sums over the wave: inside rows of 16 lanes, then the rows' last lanes onto the rows after
  auto wave_scan = [&](int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31 to rows 2 and 3
    return v;
  };
  if (B <= 64) {
    int pages = 0, tail = 0;
    const bool bad = lane < B && !dec_seq(a, d, lane, pages, tail);
    const int incl = wave_scan(pages);
    if (lane < B) {
      P.pre[lane + 1] = incl;
      P.tail[lane] = (unsigned char)tail;
    }
    if (lane == 0) P.pre[0] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int total = __builtin_amdgcn_readlane(incl, 63);
    most = pages;
    return __any(bad) ? -1 : total;
  }
  if (tid == 0) { P.err = 0; P.pre[0] = 0; P.over = 0; }
  __syncthreads();
  int carry = 0;
  most = 0;
#pragma unroll
  for (int c = 0; c < kDecPlanChunks; ++c) {
    if (c * kThreads >= B) break;                   // uniform
    const int b = c * kThreads + tid;
    int pages = 0, tail = 0;
    const bool bad = b < B && !dec_seq(a, d, b, pages, tail);
    most = max(most, pages);
    const int incl = wave_scan(pages);
    if (lane == 63) P.wsum[wv] = incl;
    if (__any(bad) && lane == 0) P.err = 1;
    __syncthreads();
    int before = carry, sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wv) before += P.wsum[w];
      sum += P.wsum[w];
    }
    if (b < B) {
      P.pre[b + 1] = before + incl;
      P.tail[b] = (unsigned char)tail;
    }
    carry += sum;
    __syncthreads();
  }
  return P.err ? -1 : carry;
}

// A place in the page list: page p (of np) of sequence b, which attends to kv keys.  All members
// are uniform across the wave.
struct PageCursor {
  int b, p, np, kv;
};

// The place of entry t (< pre[B]) of the list: the sequence is found by counting prefix sums with
// ballots (64 evenly spaced probes, then the gap between two).
__device__ __forceinline__ PageCursor locate(const DecPlanLds& P, int t, int B) {
  const int lane = threadIdx.x & 63;
  const int gap = (B + 63) / 64;
  const int blk = __popcll(__ballot(lane * gap < B && P.pre[min(lane * gap, B)] <= t)) - 1;
  int b = blk * gap;
  if (gap > 1) {
    const int i1 = b + 1 + lane;
    b += __popcll(__ballot(lane < gap - 1 && i1 < B && P.pre[min(i1, B)] <= t));
  }
  b = uni(b);
  const int first = uni(P.pre[b]);
  const int np = uni(P.pre[b + 1]) - first;
  return PageCursor{b, t - first, np, (np - 1) * kPage + uni(P.tail[b]) + 1};
}

// The next entry (never called on the list's last one).
__device__ __forceinline__ void advance(const DecPlanLds& P, PageCursor& c) {
  if (++c.p < c.np) return;
  c.p = 0;
  ++c.b;
  c.np = uni(P.pre[c.b + 1]) - uni(P.pre[c.b]);
  c.kv = (c.np - 1) * kPage + uni(P.tail[c.b]) + 1;
}

// Whether no sequence holds more than `limit` pages, `most` being decode_plan's: called once, by all
// threads.
__device__ __forceinline__ bool all_within(DecPlanLds& P, int B, int most, int limit) {
  const bool over = __any(most > limit);
  if (B <= 64) return !over;
  if (over && (threadIdx.x & 63) == 0) P.over = 1;
  __syncthreads();
  return P.over == 0;
}

// The cut of the page list.  A workgroup takes `heads` kv-heads (a power of two up to 8 that
// divides H) and one of n_runs runs of 8 / heads consecutive shares; the first `more` shares hold
// len + 1 entries, the others len.  Several heads per workgroup read the adjacent blocks of a page
// together, which HBM serves faster (2% of a share's time at 8 heads, 9% at 64).  But then every
// share's end cuts a pair between workgroups, and the last merges take longer the more pieces a pair
// is cut into.  So workgroups take several heads if the longest pair's pieces, longest / len, are few
// for the share's length: kDecPieceCost * longest / len <= len.  Measured (us a call with one head
// and with several; G = 4, G = 1 above 16 kv-heads; pages per share, pieces of the longest pair):
//   several are faster: 64 sequences of 2K-16K tokens, 8 kv-heads (144, 7) 363 and 355; 32 of 400-1600,
//     64 kv-heads (62, 1.6) 178 and 163; the same at 40 (39, 2.6) 110 and 107; 64 of 100-400, 64 kv-heads
//     (31, 1) 95.8 and 89.1; 256 of 1K-8K, 2 kv-heads (70, 7) 191 and 186;
//   one is faster: 48 of 2K-6K, 8 kv-heads (47, 8) 124 and 130; 32 of them (31, 12) 87 and 100; 16 of
//     2K-30K (64, 29) 171 and 188; 8 of 4K-16K, 16 kv-heads (39, 25) 116 and 135; 32 of 500-2000, 16
//     kv-heads (19, 6) 59 and 66; 200 of 500-2000, 4 kv-heads (30, 4) 89.5 and 90.1.
struct DecShares {
  int heads, n_runs, len, more;
  __device__ __forceinline__ DecShares(DecPlanLds& P, int pages, int most, const DecPlanArgs& d) {
    // which form and how many runs: any wave and workgroup finds the same, exact quotients are not needed
    const int len_heads = min((int)((float)pages * d.inv_shares_heads), 1 << 15);
    const int longest = len_heads * len_heads / kDecPieceCost;            // at most, for several heads
    if (d.heads > 1 && (long long)longest * d.batch >= pages && all_within(P, d.batch, most, longest)) {
      heads = d.heads;
      n_runs = d.runs_heads;
    } else {
      heads = 1;
      // Long sequences in few pairs take somewhat longer runs, so that a pair is not merged from 100
      // pieces: three of 5-20K tokens on one kv-head 22.0 us a call with kDecMinPages alone, 19.4 so.
      const int least = kDecMinPages + (int)((float)pages * d.inv_64_seqs);
      n_runs = max(1, min(d.runs_one, (int)((float)pages * __builtin_amdgcn_rcpf((float)least))));
    }
    const int n = n_runs * subs();
    len = (int)((unsigned)pages / (unsigned)n);
    more = pages - len * n;
  }
  __device__ __forceinline__ int subs() const { return kWaves / heads; }   // shares per run
  __device__ __forceinline__ int begin(int share) const { return share * len + min(share, more); }
  __device__ __forceinline__ int run_of(int t) const {                     // the run that holds entry t
    const int big = more * (len + 1);
    const int share = t < big ? (unsigned)t / (unsigned)(len + 1) : more + (unsigned)(t - big) / (unsigned)max(len, 1);
    return (unsigned)share / (unsigned)subs();
  }
};

// A wave's partials at the end of its share, in the space of its own page stages: [0] the first
// pair's, [1] the last one's.
template <int D> struct ShareEnd {
  float o[2][8][D];
  float ml[2][8][2];
};
// What they are of: the sequences of the first pair (< 0: none) and the last one, whether the last
// one started before the share, and whether the share holds pages at all.
struct SharePairs {
  int first_b, last_b, before, used;
};
// A pair cut by the workgroup's boundaries: its sequence (< 0: none), first run, runs, first slot.
struct CutPair {
  int b, x0, n, slot0;
};

// Two adjacent floats as one device-scope access: stores are written through to the level where
// every XCD reads them, loads do not hit stale cache lines.
__device__ __forceinline__ void st_dev2(float* p, float x, float y) {
  const unsigned long long v = (unsigned long long)__builtin_bit_cast(unsigned, x) |
                               ((unsigned long long)__builtin_bit_cast(unsigned, y) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ld_dev2(const float* p, float& x, float& y) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  x = __builtin_bit_cast(float, (unsigned)v);
  y = __builtin_bit_cast(float, (unsigned)(v >> 32));
}

// Merge of a cut pair (kv-head g) from its partials, in the workgroup that counted itself in last:
//   o = sum_s 2^(m_s - m*) o~_s / sum_s 2^(m_s - m*) l_s,   lse = (m* + log2 l*) ln 2.
// A lane takes D/16 dims of a q-head and the (m, l) of that head (4 heads a pass), up to kMergeBlock
// partials in flight at a time and no load beyond the pair's own (one sequence of 2732 keys, 10
// partials a pair: 13.8 us a call with blocks of 8, 13.15 with 12, 13.2 with 16; with the last
// partial loaded again to fill every block, 512 sequences of 2-3 partials took 195-200 us, now 190).
constexpr int kMergeBlock = 12;

template <int D>
__device__ __forceinline__ void merge_pair(const AttnArgs& a, const CutPair& c, int g, int stride, int max_dec, int pass) {
  constexpr int U = kMergeBlock, PER = D / 16;
  const int G = a.group, H_q = a.num_q_heads;
  const int ns = uni(c.n);
  const int lane = threadIdx.x & 63, head = 4 * pass + lane / 16, dim = lane % 16 * PER;
  if (head >= G) return;
  float M = -INFINITY, L = 0.f, acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.f;
#pragma unroll 1
  for (int s0 = 0; s0 < ns; s0 += U) {
    float v[U][PER], m[U], l[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      m[u] = -INFINITY;
      if (s0 + u < ns) {                            // uniform
        const int s = s0 + u;
        const size_t slot = ((size_t)g * max_dec + (s == 0 ? c.slot0 : stride * (c.x0 + s))) * G + head;
        ld_dev2(&a.part_ml[2 * slot], m[u], l[u]);
#pragma unroll
        for (int i = 0; i < PER; i += 2) ld_dev2(&a.part_o[slot * D + dim + i], v[u][i], v[u][i + 1]);
      }
    }
    float M_new = M;
#pragma unroll
    for (int u = 0; u < U; ++u) M_new = fmaxf(M_new, m[u]);
    const float alpha = s0 == 0 ? 0.f : fexp2(M - M_new);
    L *= alpha;
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < ns) {                            // uniform
        const float f = fexp2(m[u] - M_new);
        L += f * l[u];
#pragma unroll
        for (int i = 0; i < PER; ++i) acc[i] += f * v[u][i];
      }
    }
    M = M_new;
  }
  const float inv = 1.0f / L;
  const size_t row = (size_t)c.b * H_q + g * G + head;
#pragma unroll
  for (int i = 0; i < PER; i += 4) {
    u32x2 pk;
    pk[0] = (uint32_t)bf16_bits(acc[i] * inv) | ((uint32_t)bf16_bits(acc[i + 1] * inv) << 16);
    pk[1] = (uint32_t)bf16_bits(acc[i + 2] * inv) | ((uint32_t)bf16_bits(acc[i + 3] * inv) << 16);
    *reinterpret_cast<u32x2*>(a.out + row * D + dim + i) = pk;
  }
  if (dim == 0 && a.lse) a.lse[row] = (M + flog2(L)) * kLn2;
}

template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 4 : 2) void decode_kernel(AttnArgs a, DecPlanArgs d) {
  using PT = PageTile<D>;
  constexpr int NW = kWaves, KB = PT::KB, MB = PT::MB;
  constexpr int QB = 8 * D * 2;                     // bytes of a group's query rows (G <= 8)
  constexpr int NQ = QB / 1024;                     // DMA instructions for them
  constexpr int PAGE_LOADS = 2 * PT::NDMA;          // DMA instructions per page
  __shared__ __attribute__((aligned(16))) char stage[NW * 2 * PT::BYTES];   // per wave: two pages
  __shared__ __attribute__((aligned(16))) char qbuf[NW * QB];
  __shared__ DecPlanLds P;
  __shared__ SharePairs ends[NW];                   // per share of the run
  __shared__ CutPair s_cut[2];                      // of the first and the second slot
  __shared__ int s_last[2][NW];
  __shared__ int progress[NW];
  static_assert(sizeof(ShareEnd<D>) <= 2 * PT::BYTES, "a wave's partials fit its stages");
  const int lane = threadIdx.x & 63, w = uni(threadIdx.x >> 6);
  const int gi = lane >> 4, hh = lane & 15;
  const int G = a.group, H = a.num_kv_heads, H_q = a.num_q_heads, B = d.batch;

  int most;
  const int total_pages = uni(decode_plan(a, d, P, most));
  if (total_pages < 0) {                            // the prologue cleared the error flag
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ws_hdr[kHdrError] = 1;
    return;
  }
  DecShares sh(P, total_pages, most, d);
  // Runs of whole sequences, as many sequences each (one, if the grid holds a workgroup for every
  // (sequence, kv-head) pair), instead of equal runs, where no run gets much longer by it: then no pair
  // is cut between workgroups, and the acknowledged stores, the count-in and the merge, which take
  // about as long as 3 more pages a wave, fall away.  us a call with equal runs and so, 32 q-heads:
  // 4 sequences of 200-400 tokens at 2 kv-heads 14.1 and 11.8; 24 of 500-1000 at 8 21.1 and 19.2; but
  // one of 770 at 4, 30 pages over its run, 11.6 and 13.0; two sequences a run, 64 of 16-64 at 8 16.0 and
  // 11.1.  The line at 28 pages more than an equal run, against 12 and 60: 32 of 200-700 at 8 16.4 / 18.6 /
  // 16.4, 128 of 100-400 at 8 30.1 / 32.1 / 30.2, 300 of 100-500 at 2 25.2 / 25.2 / 26.2, 24 of 500-1200
  // at 8 22.0 / 22.1 / 21.1.  It needs no partial slots: with short sequences the workspace holds one
  // per sequence, which allows equal runs for half of them only.
  auto whole_begin = [&](int run) { return run * d.whole_seqs + min(run, d.whole_more); };
  // (up to 64 sequences every wave holds all lengths, and one that is too much by itself is seen there)
  bool whole_runs = sh.heads == 1 && !(B <= 64 && __any((most - kDecWholePages) * sh.n_runs > total_pages));
  if (whole_runs && (B > 64 || d.runs_whole < B)) {
    bool over = false;
#pragma unroll 1
    for (int i = lane; i < d.runs_whole; i += 64) {
      const int pages = P.pre[whole_begin(i + 1)] - P.pre[whole_begin(i)];
      over |= (long long)(pages - kDecWholePages) * sh.n_runs > total_pages;
    }
    whole_runs = !__any(over);
  }
  if (whole_runs) sh.n_runs = d.runs_whole;
  const int n_blk = (H + sh.heads - 1) / sh.heads;  // head blocks
  if ((int)blockIdx.x >= sh.n_runs * n_blk) return;
  // Run x of a head block is workgroup x n_blk + (block - x) mod n_blk: the blocks of a run start
  // together, and every XCD (workgroup mod 8) sees all of them.
  const int x = blockIdx.x / n_blk;
  // The last block overlaps the one before if the kv-heads don't divide: the waves of its first `dup`
  // kv-heads go along, so that all keep pace, but read one page again and again and leave no results.
  const int blk0 = (blockIdx.x + x) % n_blk * sh.heads;
  const int g0 = min(blk0, H - sh.heads), dup = blk0 - g0;
  const int sub = w / sh.heads, j_w = w % sh.heads, g = g0 + j_w;
  const bool head_ok = hh < G && j_w >= dup;
  const int pages_seen = j_w < dup ? 1 : a.num_pages;
  int run0, t0, n;                                  // the run's first entry; the wave's share
  if (whole_runs) {
    run0 = uni(P.pre[whole_begin(x)]);
    const int len = uni(P.pre[whole_begin(x + 1)]) - run0, q = len / NW, r = len % NW;
    t0 = run0 + w * q + min(w, r);
    n = q + (w < r);
  } else {
    const int share = x * sh.subs() + sub;
    run0 = sh.begin(x * sh.subs());
    t0 = sh.begin(share);
    n = sh.begin(share + 1) - t0;
  }
  // partial slots and counters of a kv-head: two slots and a counter per run, or a slot per run,
  // and a slot and a counter per sequence, if that is fewer
  const bool per_pair = B < sh.n_runs;
  const int slot_stride = per_pair ? 1 : 2;

  // State of the current pair, and of the first pair if the share only holds its end.
  f32x4 oacc[MB], o_first[MB];
  float m_run = -INFINITY, l_run = 0.f, m_first = -INFINITY, l_first = 0.f;
  int first_b = -1;                                 // the sequence of o_first
  bool whole = false;                               // the current pair started inside this share
  PageCursor cur{-1, 0, 1, 1};
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) oacc[mb] = o_first[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

  char* const st = stage + w * 2 * PT::BYTES;
  if (n > 0) {
    char* const qb = qbuf + w * QB;
    const ConstI32Ptr bt = (ConstI32Ptr)a.block_table;
    auto raw_id = [&](const PageCursor& c) { return bt[(size_t)c.b * a.bt_stride + c.p]; };
    // the group's query rows of a pair (rows past the group repeat its last one)
    auto issue_q = [&](const PageCursor& c) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int r = min((i * 64 + lane) / PT::CPR, G - 1);
        lds_dma16_untracked(a.q + ((size_t)c.b * H_q + g * G + r) * D + (lane % PT::CPR) * 8, qb + i * 1024);
      }
    };
    const PageCopies<D> copies(lane);
    // a page's copies: a sequence's last page may hold the new row and rows past the end; every other
    // one is two whole blocks
    auto issue_page = [&](const PageCursor& c, int raw, char* dst) {
      const int phys = clamp_page(raw, pages_seen);
      if (c.p == c.np - 1) {
        NewRow nr{-1, 0, a.k_pool, a.v_pool};       // no new row (valid pointers, never selected)
        if (a.k_new) {
          const size_t row = ((size_t)c.b * H + g) * D;
          nr = NewRow{c.p, (c.kv - 1) % kPage, a.k_new + row, a.v_new + row};
        }
        decode_issue<D, true>(a, phys, c.p, g, c.kv, dst, nr);
      } else {
        const size_t blk = ((size_t)phys * H + g) * (size_t)(kPage * D);
        copies.issue(a.k_pool + blk, a.v_pool + blk, dst);
      }
    };
    bf16x8 qop[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) qop[kb] = zero_bf16x8();
    cur = locate(P, t0, B);
    PageCursor nxt = cur;
    int raw_cur = raw_id(cur), raw_nxt = 0;
    issue_q(cur);
    issue_page(cur, raw_cur, st);
    if (n > 1) {
      advance(P, nxt);
      raw_nxt = raw_id(nxt);
    }
    // step k: the copies of page k + 1 go out, then page k (and its pair's query rows) is waited for
    // and attended.  fresh: page k is the first of its pair in this share; q_sent: its query rows
    // are on their way (they go out behind the pair's first page, a step ahead, unless the one
    // before was itself the first page of its pair and still needs the query buffer).
    bool fresh = true, q_sent = true;
    int buf = 0;
    for (int k = 0; k < n; ++k) {
      // A SIMD's two waves (w and w ^ 4) keep pace: the one behind issues first.  Left alone, the
      // older one always does: waves 4-7 took 17% longer than waves 0-3.
      if (lane == 0) *(volatile int*)&progress[w] = k;
      if (uni(*(volatile int*)&progress[w ^ 4]) > k) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
      // Waves of several heads go page by page together, so that the adjacent blocks of a page are
      // read together (without this barrier the 355 us above are 362, with it every 4th page 358).
      if (sh.heads > 1 && k < sh.len) __asm__ volatile("s_barrier" ::: "memory");
      if (fresh && !q_sent) issue_q(cur);
      PageCursor nn = nxt;
      int raw_nn = 0;
      if (k + 1 < n) {
        const bool nxt_fresh = nxt.p == 0;
        issue_page(nxt, raw_nxt, st + (buf ^ PT::BYTES));
        if (k + 2 < n) {
          advance(P, nn);
          raw_nn = raw_id(nn);
        }
        q_sent = nxt_fresh && !fresh;
        if (q_sent) {
          issue_q(nxt);
          __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"(PAGE_LOADS + NQ) : "memory");
        } else {
          __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"(PAGE_LOADS) : "memory");
        }
      } else {
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      if (fresh) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const bf16x8 q = *reinterpret_cast<const bf16x8*>(qb + (hh & 7) * (D * 2) + (4 * kb + gi) * 16);
          qop[kb] = head_ok ? q : zero_bf16x8();
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) oacc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run = -INFINITY;
        l_run = 0.f;
        whole = cur.p == 0;
      }
      decode_consume<D, true>(cur.p, cur.kv, qop, oacc, m_run, l_run, a.scale_log2, st + buf);
      const bool ends_here = cur.p == cur.np - 1;
      if (ends_here && a.k_new) {
        // the new token's row goes into the pools from the stage (no wave reads it from there; a
        // page id out of range is skipped, as pearl_kv_append does)
        const int r = (cur.kv - 1) % kPage;
        const int c = lane % PT::CPR;
        const bool is_v = lane >= PT::CPR;
        const u32x4 y = *reinterpret_cast<const u32x4*>(
            st + buf + (is_v ? PT::TBYTES + r * PT::ROWB + ((c ^ PT::vswz(r)) << 4) : PT::koff(r, c)));
        if (lane < 2 * PT::CPR && j_w >= dup && raw_cur >= 0 && raw_cur < a.num_pages) {
          const size_t dst = (((size_t)raw_cur * H + g) * kPage + r) * D + 8 * c;
          *reinterpret_cast<u32x4*>((is_v ? a.v_pool_w : a.k_pool_w) + dst) = y;
        }
      }
      if (ends_here) {
        // each head's four lane groups hold different keys: sum their l
        l_run += __shfl_xor(l_run, 16);
        l_run += __shfl_xor(l_run, 32);
        if (whole) {
          if (head_ok) {
            const size_t row = (size_t)cur.b * H_q + g * G + hh;
            uint16_t* orow = a.out + row * D + 4 * gi;
            const float inv = 1.0f / l_run;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
              u32x2 pk;
              pk[0] = (uint32_t)bf16_bits(oacc[mb][0] * inv) | ((uint32_t)bf16_bits(oacc[mb][1] * inv) << 16);
              pk[1] = (uint32_t)bf16_bits(oacc[mb][2] * inv) | ((uint32_t)bf16_bits(oacc[mb][3] * inv) << 16);
              *reinterpret_cast<u32x2*>(orow + 16 * mb) = pk;
            }
            if (gi == 0 && a.lse) a.lse[row] = (m_run + flog2(l_run)) * kLn2;
          }
        } else {                                    // only the first pair can have started earlier
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) o_first[mb] = oacc[mb];
          m_first = m_run;
          l_first = l_run;
          first_b = cur.b;
        }
      }
      fresh = ends_here;
      if (k + 1 == n) {
        if (ends_here) cur.b = -1;                  // the share ends with the pair's end
        break;
      }
      cur = nxt;
      raw_cur = raw_nxt;
      nxt = nn;
      raw_nxt = raw_nn;
      buf ^= PT::BYTES;
    }
    if (cur.b >= 0) {
      l_run += __shfl_xor(l_run, 16);
      l_run += __shfl_xor(l_run, 32);
    }
  }

  // the waves' partials, merged per pair through LDS
  {
    ShareEnd<D>& E = *reinterpret_cast<ShareEnd<D>*>(st);
    if (head_ok) {
      if (first_b >= 0) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(&E.o[0][hh][16 * mb + 4 * gi]) = o_first[mb];
        if (gi == 0) { E.ml[0][hh][0] = m_first; E.ml[0][hh][1] = l_first; }
      }
      if (cur.b >= 0) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(&E.o[1][hh][16 * mb + 4 * gi]) = oacc[mb];
        if (gi == 0) { E.ml[1][hh][0] = m_run; E.ml[1][hh][1] = l_run; }
      }
    }
    if (lane == 0) ends[sub] = SharePairs{first_b, cur.b, !whole, n > 0};   // alike for all heads
    if (threadIdx.x < 2) s_cut[threadIdx.x].b = -1;
  }
  // a barrier without the release fence of __syncthreads: output stores stay in flight
  __builtin_amdgcn_s_waitcnt(PEARL_LGKMCNT0);
  __asm__ volatile("s_barrier" ::: "memory");
  // A pair's partials form a chain: it starts in the share the pair starts in (or in the run's first
  // share), goes on through the last-pair partials of the following shares while the pair goes
  // on, and closes with the first-pair partial of the share the pair ends in.  Bit q of the masks
  // below is share q's.
  {
    const int subs = sh.subs();
    const SharePairs e = ends[lane & (NW - 1)];
    const unsigned used = (unsigned)__ballot(lane < subs && e.used);
    const unsigned has_first = (unsigned)__ballot(lane < subs && e.first_b >= 0);
    // bits 0..7: chains that start with share q's last pair; bit 8: the first share's first pair
    unsigned todo = (unsigned)__ballot(lane < subs && e.last_b >= 0 && (!e.before || lane == 0)) |
                    ((has_first & 1u) << NW);
    const int rows = sh.heads * G;                  // q-heads of the workgroup
    while (todo) {
      const int q0 = __builtin_ctz(todo);
      todo &= todo - 1;
      const bool is_first = q0 == NW;
      const int qb = is_first ? 0 : q0;
      const unsigned after = is_first ? 0u : ~0u << (q0 + 1);
      const unsigned close = has_first & after;     // its lowest bit: the share that closes the chain
      const unsigned mid = is_first ? 0u : (used & after & ((close & -close) - 1u)) | (1u << q0);
      const int q_close = is_first ? 0 : (close ? __builtin_ctz(close) : -1);
      const int b = __builtin_amdgcn_readlane(is_first ? e.first_b : e.last_b, qb);
      const bool before = is_first || __builtin_amdgcn_readlane(e.before, qb);
      const bool cut = before || q_close < 0;       // other workgroups hold parts of it
      const int pu = uni(P.pre[b]);                 // the pair's first entry
      const int second = pu > run0;
      const int slot2 = per_pair ? sh.n_runs + b : 2 * x + 1;   // the run's second slot
      for (int t = threadIdx.x + dup * G * (D / 2); t < rows * (D / 2); t += kThreads) {
        const int r = t / (D / 2), dim = 2 * (t - r * (D / 2));
        const int j = r / G, head = r - j * G;      // kv-head of the workgroup, q-head of the group
        float M = -INFINITY, L = 0.f, o0 = 0.f, o1 = 0.f;
        auto add = [&](int q, int which) {
          const ShareEnd<D>& E = *reinterpret_cast<const ShareEnd<D>*>(stage + (q * sh.heads + j) * 2 * PT::BYTES);
          const float m = E.ml[which][head][0], l = E.ml[which][head][1];
          const float M_new = fmaxf(M, m);
          const float fa = M == -INFINITY ? 0.f : fexp2(M - M_new), fb = fexp2(m - M_new);
          L = fa * L + fb * l;
          o0 = fa * o0 + fb * E.o[which][head][dim];
          o1 = fa * o1 + fb * E.o[which][head][dim + 1];
          M = M_new;
        };
        for (unsigned rest = mid; rest; rest &= rest - 1) add(__builtin_ctz(rest), 1);
        if (q_close >= 0) add(q_close, 0);
        if (!cut) {
          const size_t row = (size_t)b * H_q + g0 * G + r;
          const float inv = 1.0f / L;
          *reinterpret_cast<uint32_t*>(a.out + row * D + dim) =
              (uint32_t)bf16_bits(o0 * inv) | ((uint32_t)bf16_bits(o1 * inv) << 16);
          if (dim == 0 && a.lse) a.lse[row] = (M + flog2(L)) * kLn2;
        } else {
          const size_t slot = ((size_t)(g0 + j) * d.max_dec + (second ? slot2 : slot_stride * x)) * G + head;
          st_dev2(&a.part_o[slot * D + dim], o0, o1);
          if (dim == 0) st_dev2(&a.part_ml[2 * slot], M, L);
        }
      }
      if (cut && threadIdx.x == 0) {
        const int x0 = sh.run_of(pu), x1 = sh.run_of(uni(P.pre[b + 1]) - 1);
        const bool at_start = pu <= sh.begin(x0 * subs);
        s_cut[second] = CutPair{b, x0, x1 - x0 + 1, at_start ? slot_stride * x0 : (per_pair ? slot2 : 2 * x0 + 1)};
      }
    }
  }
  // Count the run in on its cut pairs once its stores are acknowledged; the last one merges.  The
  // counter of a pair is its sequence's, or (of as many counters as runs) that of the run it starts
  // in: at most one pair goes on past a run's end.
  __builtin_amdgcn_s_waitcnt(PEARL_VMCNT(0));
  __syncthreads();
  const int task = threadIdx.x;                     // (slot kind, kv-head of the workgroup)
  if (task < 2 * sh.heads) {
    const int j = task >> 1;
    const CutPair c = s_cut[task & 1];
    int last = 0;
    if (c.b >= 0 && j >= dup) {
      const int ctr = per_pair ? (g0 + j) * B + c.b : (g0 + j) * sh.n_runs + c.x0;
      last = __hip_atomic_fetch_add(&a.split_cnt[ctr], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == c.n - 1;
    }
    s_last[task & 1][j] = last;
  }
  __syncthreads();
  const int passes = (G + 3) / 4;
#pragma unroll 1
  for (int t = w; t < 2 * sh.heads * passes; t += NW) {
    const int pair = t / passes;
    if (s_last[pair & 1][pair >> 1])
      merge_pair<D>(a, s_cut[pair & 1], g0 + (pair >> 1), slot_stride, d.max_dec, t - pair * passes);
  }
}

// Zeroes what the decode kernel needs zeroed: the workspace header (error flag, the zero block)
// and the arrival counters.  A kernel, not a memset, so it can be captured.
__global__ __launch_bounds__(256) void decode_prologue_kernel(int32_t* hdr, int32_t* split_cnt, int n_cnt) {
  for (int i = threadIdx.x; i < n_cnt; i += 256) split_cnt[i] = 0;
  if (threadIdx.x < kHdrWords) hdr[threadIdx.x] = 0;
}

// ------------------------------------------------------------------------------------------------
// Split merge: one wave per (sequence, q-head) with more than one split.  The maximum of the
// split maxima is found with a wavefront shuffle reduction; then
//   o = sum_s 2^(m_s - m*) o~_s / sum_s 2^(m_s - m*) l_s,   lse = (m* + log2 l*) ln 2.
// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void merge_kernel(AttnArgs a, int batch) {
  const int lane = threadIdx.x & 63;
  const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int H_q = a.num_q_heads;
  if (wid >= batch * H_q) return;
  const int b = wid / H_q, h = wid - (wid / H_q) * H_q;
  // three independent reads (the record and base of a sequence the planner skipped are read but
  // not used)
  const int err = a.ws_hdr[kHdrError];
  const SeqInfo si = a.seqinfo[b];
  const size_t base = (size_t)a.split_base[b];
  const int ns = si.kind >> 4;
  if (err != 0 || (si.kind & 15) != kSeqDecode || ns <= 1) return;
  float M = -INFINITY;
  for (int s = lane; s < ns; s += 64) M = fmaxf(M, a.part_ml[2 * ((base + s) * H_q + h)]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  constexpr int PER = D / 64;
  constexpr int U = 8;                              // splits whose o~ loads are in flight together
  float acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.f;
  float L = 0.f;
  for (int s0 = 0; s0 < ns; s0 += 64) {
    const int cnt = min(64, ns - s0);
    // lane j computes split s0 + j's weight 2^(m - M) and its share of the sum
    float f = 0.f;
    if (lane < cnt) {
      const size_t pidx = (base + s0 + lane) * H_q + h;
      f = fexp2(a.part_ml[2 * pidx] - M);
      L += f * a.part_ml[2 * pidx + 1];
    }
    for (int j = 0; j < cnt; j += U) {
      float v[U][PER], fj[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int jj = min(j + u, cnt - 1);       // past the end: reload the last split, weight 0
        const float w = __shfl(f, jj);
        fj[u] = j + u < cnt ? w : 0.f;
        const size_t pidx = (base + s0 + jj) * H_q + h;
#pragma unroll
        for (int i = 0; i < PER; ++i) v[u][i] = a.part_o[pidx * D + lane * PER + i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < PER; ++i) acc[i] += fj[u] * v[u][i];
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) L += __shfl_xor(L, off);
  const float inv = 1.0f / L;
  uint16_t* orow = a.out + ((size_t)si.q_start * H_q + h) * D + lane * PER;
#pragma unroll
  for (int i = 0; i < PER; ++i) orow[i] = bf16_bits(acc[i] * inv);
  if (lane == 0 && a.lse) a.lse[(size_t)si.q_start * H_q + h] = (M + flog2(L)) * kLn2;
}

// ------------------------------------------------------------------------------------------------
// Merge of split prefill tiles, grid-stride over the (job, kv-head, tile row) the planner recorded:
// D / 4 lanes per row, 4 dims each, kPreMergeBlock splits in flight at a time.  Same combination as
// the decode merge, over the tile's splits.  It reads 4 D bytes per row and split once; few loads in
// flight per row, so several rows share a wave.  2, 4 and 8 splits in flight are within 2% of a call
// (append, plan, attention, merge): eight turns of 64-300 tokens on 4-8K contexts 183 / 183 / 186 us, 16
// of 100-300 on 4-6K at d = 64 129 / 130 / 131.
// ------------------------------------------------------------------------------------------------
constexpr int kMergeMaxBlocks = 2048;
constexpr int kPreMergeBlock = 4;

template <int D>
__global__ __launch_bounds__(256) void merge_prefill_kernel(AttnArgs a) {
  constexpr int LPR = D / 4, RPB = 256 / LPR, U = kPreMergeBlock;   // lanes per row, rows per workgroup
  const int err = a.ws_hdr[kHdrError], jobs = a.ws_hdr[kHdrNumPreJobs];
  const int H_kv = a.num_kv_heads, H_q = a.num_q_heads, G = a.group, T = a.tokens_per_tile;
  const int total = err != 0 ? 0 : jobs * H_kv * kRowsPerTile;
  const int dim = threadIdx.x % LPR * 4;
  for (int r = blockIdx.x * RPB + threadIdx.x / LPR; r < total; r += gridDim.x * RPB) {
    const int rho = r % kRowsPerTile, jg = r / kRowsPerTile;
    const int g = jg % H_kv, j = jg / H_kv;
    const int4 job = a.pre_jobs[j];                  // (sequence, tile, first slot, splits)
    const SeqInfo si = a.seqinfo[job.x];
    const int tok = job.y * T + rho / G;
    if (tok >= si.q_len) continue;
    const int nt = (si.q_len + T - 1) / T;           // slots from one split of the tile to the next
    const int ns = job.w;
    float M = -INFINITY, L = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s0 = 0; s0 < ns; s0 += U) {
      float m[U], l[U];
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int sp = min(s0 + u, ns - 1);          // past the end: the last split, weight 0
        const size_t prow = (size_t)((job.z + sp * nt) * H_kv + g) * kRowsPerTile + rho;
        m[u] = a.part_pre_ml[2 * prow];
        l[u] = a.part_pre_ml[2 * prow + 1];
        v[u] = *reinterpret_cast<const f32x4*>(a.part_pre_o + prow * D + dim);
      }
      float M_new = M;
#pragma unroll
      for (int u = 0; u < U; ++u) M_new = fmaxf(M_new, m[u]);
      const float alpha = s0 == 0 ? 0.f : fexp2(M - M_new);
      L *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= ns) break;
        const float f = fexp2(m[u] - M_new);
        L += f * l[u];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += f * v[u][i];
      }
      M = M_new;
    }
    const float inv = 1.0f / L;
    const size_t orow = (size_t)(si.q_start + tok) * H_q + g * G + rho % G;
    u32x2 pk;
    pk[0] = (uint32_t)bf16_bits(acc[0] * inv) | ((uint32_t)bf16_bits(acc[1] * inv) << 16);
    pk[1] = (uint32_t)bf16_bits(acc[2] * inv) | ((uint32_t)bf16_bits(acc[3] * inv) << 16);
    *reinterpret_cast<u32x2*>(a.out + orow * D + dim) = pk;
    if (dim == 0 && a.lse) a.lse[orow] = (M + flog2(L)) * kLn2;
  }
}

// ------------------------------------------------------------------------------------------------
// Device memory of the allocation-free decode entry point (pearl_attn_decode_static): the
// workspace of one call, one array per device for the life of the process.  Host code never uses
// the array's name as an address: the device address comes from hipGetSymbolAddress, taken once
// per device with that device current.
// ------------------------------------------------------------------------------------------------
static __device__ __align__(256) char scratch[kStaticScratchBytes];

// ------------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------------
namespace {
// Launch parameters per device (compute units, occupancy per kernel), queried on the first call
// that runs on the device.  Initialisation is guarded so concurrent first calls are safe.
struct DevCache {
  std::atomic<int> ready{0};
  int num_cu = 0;
  int occ[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};   // [D == 128][kinds]
  int occ_dec[2] = {0, 0};                        // decode_kernel, [D == 128]
  void* scratch = nullptr;                        // device address of this device's scratch array
  hipError_t scratch_err = hipSuccess;
};

template <int D, int K>
int occupancy_of() {
  int o = 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, attn_kernel<D, K>, KernelCfg<D, K>::NT, 0) != hipSuccess || o < 1) o = 1;
  return o;
}

template <int D>
int occupancy_of_dec() {
  int o = 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, decode_kernel<D>, kThreads, 0) != hipSuccess || o < 1) o = 1;
  return o;
}

void fill_cache(DevCache& c, int dev) {
  hipDeviceProp_t prop;
  int ncu = 256;
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0) ncu = prop.multiProcessorCount;
  c.occ[0][1] = occupancy_of<64, 1>(); c.occ[0][2] = occupancy_of<64, 2>(); c.occ[0][3] = occupancy_of<64, 3>();
  c.occ[1][1] = occupancy_of<128, 1>(); c.occ[1][2] = occupancy_of<128, 2>(); c.occ[1][3] = occupancy_of<128, 3>();
  c.occ_dec[0] = occupancy_of_dec<64>(); c.occ_dec[1] = occupancy_of_dec<128>();
  c.num_cu = ncu;
  void* p = nullptr;
  c.scratch_err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  c.scratch = c.scratch_err == hipSuccess ? p : nullptr;
}

constexpr int kCachedDevices = 64;
DevCache g_cache[kCachedDevices];
std::mutex g_cache_mutex;

const DevCache& dev_cache() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
  if (dev >= kCachedDevices) {                   // beyond the cache: query every time
    thread_local DevCache t;
    fill_cache(t, dev);
    return t;
  }
  DevCache& c = g_cache[dev];
  if (!c.ready.load(std::memory_order_acquire)) {
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    if (!c.ready.load(std::memory_order_relaxed)) {
      fill_cache(c, dev);
      c.ready.store(1, std::memory_order_release);
    }
  }
  return c;
}
}  // namespace

int device_num_cu() { return dev_cache().num_cu; }

void* static_scratch(hipError_t* err) {
  const DevCache& c = dev_cache();
  if (err) *err = c.scratch_err;
  return c.scratch;
}

int attention_grid(int head_dim, int kinds) {
  const DevCache& c = dev_cache();
  return c.num_cu * c.occ[head_dim == 128 ? 1 : 0][kinds];
}

hipError_t launch_plan(const PlanParams& p, const int32_t* ctx_lens, const int32_t* cu_q_lens,
                       void* workspace, const WsLayout& lay, hipStream_t stream) {
  char* ws = static_cast<char*>(workspace);
  auto kernel = p.mode == kModePrefill ? plan_kernel<kModePrefill> : p.mode == kModeDecode ? plan_kernel<kModeDecode>
                                                                                           : plan_kernel<kModeMixed>;
  hipLaunchKernelGGL(kernel, dim3(1), dim3(kPlanThreads), 0, stream, p, ctx_lens, cu_q_lens,
                     reinterpret_cast<int32_t*>(ws + lay.hdr), reinterpret_cast<SeqInfo*>(ws + lay.seqinfo),
                     reinterpret_cast<int32_t*>(ws + lay.split_base), reinterpret_cast<int2*>(ws + lay.entries),
                     reinterpret_cast<int4*>(ws + lay.pre_jobs));
  return hipGetLastError();
}

hipError_t launch_attention(const AttnArgs& a, int head_dim, int kinds, int64_t max_items, int max_pre,
                            hipStream_t stream) {
  if (max_items <= 0) return hipSuccess;
  if (kinds < 1 || kinds > 3) return hipErrorInvalidValue;
  const DevCache& c = dev_cache();
  const int occ = c.occ[head_dim == 128 ? 1 : 0][kinds];
  int64_t grid = (int64_t)c.num_cu * occ;
  if (grid > max_items) grid = max_items;
  const dim3 g((unsigned)grid);
  if (head_dim == 64) {
    if (kinds == 1) hipLaunchKernelGGL((attn_kernel<64, 1>), g, dim3(KernelCfg<64, 1>::NT), 0, stream, a, max_pre);
    else if (kinds == 2) hipLaunchKernelGGL((attn_kernel<64, 2>), g, dim3(KernelCfg<64, 2>::NT), 0, stream, a, max_pre);
    else hipLaunchKernelGGL((attn_kernel<64, 3>), g, dim3(KernelCfg<64, 3>::NT), 0, stream, a, max_pre);
  } else {
    if (kinds == 1) hipLaunchKernelGGL((attn_kernel<128, 1>), g, dim3(KernelCfg<128, 1>::NT), 0, stream, a, max_pre);
    else if (kinds == 2) hipLaunchKernelGGL((attn_kernel<128, 2>), g, dim3(KernelCfg<128, 2>::NT), 0, stream, a, max_pre);
    else hipLaunchKernelGGL((attn_kernel<128, 3>), g, dim3(KernelCfg<128, 3>::NT), 0, stream, a, max_pre);
  }
  return hipGetLastError();
}

int decode_grid(int head_dim) {
  const DevCache& c = dev_cache();
  return c.num_cu * c.occ_dec[head_dim == 128 ? 1 : 0];
}

void set_decode_runs(DecPlanArgs& d, int num_kv_heads, int grid) {
  // a run leaves at most two partials per head, the second ones also at most one per sequence
  const int cap = std::max(1, std::max(d.max_dec / 2, d.max_dec - d.batch));
  // a workgroup per run if they are all resident; with more kv-heads than that, runs for several rounds
  const int per_head = std::max(1, (num_kv_heads <= grid ? grid : kDecRounds * grid) / num_kv_heads);
  d.runs_one = std::min(per_head, cap);
  d.runs_whole = std::min(per_head, d.batch);
  d.whole_seqs = d.batch / d.runs_whole;
  d.whole_more = d.batch % d.runs_whole;
  d.heads = std::min(num_kv_heads & -num_kv_heads, kWaves);
  // Above 64 kv-heads, where adjacent reads matter most, blocks of 8 with a partial last one (us a call
  // with a kv-head per workgroup and so, of 400-1600 tokens: 8 sequences at 255 kv-heads 193 and 173, 15
  // at 129 181 and 168, 28 at 71 176 and 166; but 40 at 31 103 and 106).
  if (d.heads < 4 && num_kv_heads > 64) d.heads = kWaves;
  const int blocks = (num_kv_heads + d.heads - 1) / d.heads;
  d.runs_heads = std::max(1, grid / blocks);
  if (8 * cap >= 7 * d.runs_heads) {                // not enough slots for a full grid of them, nearly
    d.runs_heads = std::min(d.runs_heads, cap);
  } else {
    d.heads = 1;
    d.runs_heads = 0;
  }
  d.inv_shares_heads = d.heads > 1 ? 1.f / (float)(kWaves / d.heads * d.runs_heads) : 0.f;
  d.inv_64_seqs = 1.f / (64.f * (float)d.batch);
  d.grid = std::max(grid, std::max(std::max(d.runs_one, d.runs_whole) * num_kv_heads, d.runs_heads * blocks));
}

hipError_t launch_decode_prologue(const AttnArgs& a, const DecPlanArgs& d, hipStream_t stream) {
  // a counter per sequence and kv-head, or per run and kv-head if that is fewer
  const int n = std::min(d.batch, std::max(d.runs_one, d.runs_heads)) * a.num_kv_heads;
  hipLaunchKernelGGL(decode_prologue_kernel, dim3(1), dim3(256), 0, stream, a.ws_hdr, a.split_cnt, n);
  return hipGetLastError();
}

hipError_t launch_decode(const AttnArgs& a, const DecPlanArgs& d, int head_dim, hipStream_t stream) {
  if (head_dim == 64)
    hipLaunchKernelGGL(decode_kernel<64>, dim3((unsigned)d.grid), dim3(kThreads), 0, stream, a, d);
  else
    hipLaunchKernelGGL(decode_kernel<128>, dim3((unsigned)d.grid), dim3(kThreads), 0, stream, a, d);
  return hipGetLastError();
}

hipError_t launch_merge(const AttnArgs& a, int head_dim, int batch, hipStream_t stream) {
  const int64_t waves = (int64_t)batch * a.num_q_heads;
  const unsigned grid = (unsigned)((waves + 3) / 4);
  if (grid == 0) return hipSuccess;
  if (head_dim == 64)
    hipLaunchKernelGGL(merge_kernel<64>, dim3(grid), dim3(256), 0, stream, a, batch);
  else
    hipLaunchKernelGGL(merge_kernel<128>, dim3(grid), dim3(256), 0, stream, a, batch);
  return hipGetLastError();
}

hipError_t launch_merge_prefill(const AttnArgs& a, int head_dim, int64_t jobs_cap, hipStream_t stream) {
  const int64_t rows = jobs_cap * a.num_kv_heads * kRowsPerTile;
  int64_t grid = rows * (head_dim / 4) / 256;
  if (grid > kMergeMaxBlocks) grid = kMergeMaxBlocks;
  if (grid <= 0) return hipSuccess;
  if (head_dim == 64)
    hipLaunchKernelGGL(merge_prefill_kernel<64>, dim3((unsigned)grid), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(merge_prefill_kernel<128>, dim3((unsigned)grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pearl
