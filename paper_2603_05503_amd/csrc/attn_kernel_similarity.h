// Spatial similarity score of attention heads (paper, Section 3.3, detection of
// spatially repetitive heads) without materialising the attention map.
// gfx950 (MI355X), bf16 in, fp32 out.
//
// The score of a head is the mean, over spatial rows, of the cosine similarity
// between the attention rows of the row's tokens and those of the matching
// tokens of its anchor row (same frame, same column), both flattened over
// (column, key).  Per token t with partner a:
//     dot[t] = sum_j P[t][j] P[a][j],  nt[t] = sum_j P[t][j]^2,  na[t] = sum_j P[a][j]^2
// and per spatial row  cos = sum_x dot / sqrt(sum_x nt * sum_x na).
//
// Main kernel: one workgroup per (batch, head, 128 lane groups).  A lane holds
// R + 1 queries - one partner and up to R tokens that share it - and makes ONE
// pass over all keys: row sums, sums of squares and the R sums of products are
// kept relative to a reference per query that is moved, and the sums rescaled,
// only when a logit leaves the safe range above it; the normalisers divide out
// at the end.  Writes the normalised triple of every token.
//
// What bounds it: the vector ALU (per logit an FMA, an exponential, two or
// three sums) beside the matrix cores, and the power both draw; where a
// workgroup has its CU to itself, the chain of one wavefront.  A token and
// its partner alone (R = 1) cost two rows of logits; tokens that share their
// partner's row cost (R + 1) / R each, and one K operand read from LDS feeds
// R + 1 MFMAs.  All quantities of a query or pair are computed by the same
// operations in the same order whatever else the lane and the wave hold, so the
// bits do not depend on how the tokens were grouped.
//
// Measured, 24 heads of 21 x 30 x 52 tokens, D = 128, five anchors, in turn on one box: 13.87 ms with every token
// beside its own partner over whole tiles and one wavefront per head in the reduction, 9.84 ms in twos, 2 % less mixed.
//
// Without groups, us with one score buffer (and before it, with whole tiles of 128 keys) -> with two: 210 units of 3840
// keys, D = 128 95 (92) -> 81, D = 64 78 (73) -> 69; 480 units 148 (156) -> 141; 1800 units of 9600 keys 1299 (1427) ->
// 1296.
//
// Grouping (similarity_group_kernel): the tokens of one column of the grid in
// consecutive spatial rows form a run while they have the same partner; a run
// is cut into groups of R, or of three and two.  Groups are appended to a list in any order.
//
// Reduction kernel: one workgroup per (batch, head) adds the triples of each spatial
// row, forms the cosine and averages over rows in a fixed order.
#pragma once
#include "attn_kernel_2wg.h"

#include <float.h>

namespace calibatt_dev {

struct SimilarityDims {
  int B, H, N, n_tok, nbq, nbk, row_len;
  float scale_log2e;
};

constexpr int SIM_BQ = 128;
constexpr int SIM_BK = 64;
constexpr int SIM_XCDS = 8;
// The tokens are grouped where the pair form has more than SIM_GROUP_TURNS units of 128 tokens per CU and a head has more
// than SIM_GROUP_TOKENS tokens.  Up to two units per CU even the best groups save a CU only one of four rows of logits,
// which a single workgroup on it takes about as long for, and the lists cost 6-10 us: 16 heads of 3840 tokens, D = 128,
// 135 us in pairs, 140 grouped; 18 heads 189 and 177.  In heads of a few units the groups save no whole unit: 200 heads of
// 384 tokens 28 us in pairs, 38 grouped; 220 heads of 640 tokens 62 and 50.
constexpr int SIM_GROUP_TURNS = 2;
constexpr int SIM_GROUP_TOKENS = 512;

// The mixed form is taken where the busiest CU has less than 96 % of the rows of the best other form to do, a row of
// threes counted 1.15 times (their partner's operand comes from LDS).  Either side, rows of the others' best and of the
// mixed form, D = 128: 24 heads of 21 x 30 x 52 tokens, five anchors, 36 and 34.2: 10.20 -> 10.01 ms (D = 64 7.49 -> 7.19);
// 18 heads of 4 x 30 x 32, five anchors, 176 -> 141 us; not taken: 12 heads of 8 x 32 x 75, four anchors, 12 and 11.7: 1.93
// and 2.02 ms.
constexpr int SIM_THREE_COST = 46, SIM_MIXED_GAIN = 96;  // tenths of a row, per cent

// ---- lists of the grouped form -------------------------------------------------------------------
// int32 words: [0..2] numbers of 2-token groups, 3-token groups and lone tokens, [4 ..] the 3-token
// groups (4 words each: partner, tokens; -1 = none), the 2-token groups (likewise) and the lone tokens,
// room for n_tok of each.  A partner that takes its own triple from this group is stored as ~partner.
// The mixed form cuts a run into threes and, at its end, up to two twos, without an empty place: its groups lie at the
// far ends of the two segments, the last one first (a run of two tokens or more leaves the room), their numbers in word 3
// and in the last word of the lone tokens.  A run of one token, which has no such cut, sets the sign of word 3.
struct SimilarityLists {
  // Rows at which a run of more than LONGEST rows ends in any case: bounds the walks below, 0.1 us a row.  The runs of a
  // video, of up to the rows of a frame, stay whole: a cut leaves single tokens, which have no place in the mixed form.
  // 630 rows of 52 tokens with one partner row, 4 heads: 1.79 ms, with walks of up to 1024 rows 1.95.
  static constexpr int LONGEST = 64, SEGMENT = 64;
  static __host__ __device__ long long bytes(int n_tok) { return 16 + 36LL * n_tok; }
  static __device__ __forceinline__ int4 *groups(int32_t *lists, int n_tok, int R) {
    return reinterpret_cast<int4 *>(lists + 4) + (R == 3 ? 0 : n_tok);
  }
  static __device__ __forceinline__ int32_t *lone(int32_t *lists, int n_tok) { return lists + 4 + 8LL * n_tok; }
  static __device__ __forceinline__ int32_t *mixed_twos(int32_t *lists, int n_tok) { return lone(lists, n_tok) + n_tok - 1; }
};

__global__ __launch_bounds__(64) void similarity_clear_kernel(int32_t *__restrict__ lists, int n_tok) {
  if (threadIdx.x < 4) lists[threadIdx.x] = 0;
  if (threadIdx.x == 4) *SimilarityLists::mixed_twos(lists, n_tok) = 0;
}

__device__ __forceinline__ int similarity_partner(const int32_t *__restrict__ partner, int t, int N) {
  const int a = partner[t];
  return a < 0 ? 0 : (a < N ? a : N - 1);
}

// One thread per token.
__global__ __launch_bounds__(256) void similarity_group_kernel(const int32_t *__restrict__ partner,
                                                               int32_t *__restrict__ lists, int N, int n_tok,
                                                               int row_len) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  const bool here = t < n_tok;
  const int a = here ? similarity_partner(partner, t, N) : -1;
  const int row = here ? t / row_len : 0;
  // The run: rows of this column around the token's with the same partner, and the partner's own row if it is one of them.
  // More than LONGEST rows or not, every token of a run finds the same.
  constexpr int LONGEST = SimilarityLists::LONGEST, SEGMENT = SimilarityLists::SEGMENT;
  int before = 0, behind = 0, next[2] = {-1, -1};  // tokens of the run that are not their own partner
  bool own = false;
  if (here) {
    const int n_rows = n_tok / row_len, segment = row / SEGMENT * SEGMENT, col = t - row * row_len;
    auto same = [&](int y) { return similarity_partner(partner, y * row_len + col, N) == a; };
    int first = row, last = row;
    while (first > 0 && row - first < LONGEST && same(first - 1)) --first;
    while (last + 1 < n_rows && (last - first < LONGEST || last + 1 < segment + SEGMENT) && same(last + 1)) ++last;
    if (last - first >= LONGEST) {
      first = max(first, segment);
      last = min(last, segment + SEGMENT - 1);
    }
    const int partner_row = a / row_len;
    own = partner_row != row && partner_row >= first && partner_row <= last && a - partner_row * row_len == col;
    before = row - first - (own && partner_row < row);
    behind = last - row - (own && partner_row > row);
    for (int i = 0, y = row; i < min(behind, 2); ++i) {
      y += own && y + 1 == partner_row ? 2 : 1;
      next[i] = y * row_len + col;
    }
  }
  // appends to a list: one atomic per wavefront
  auto append = [&](bool mine, int32_t *counter) {
    const unsigned long long who = __ballot(mine);
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (who && lane == __ffsll(who) - 1) base = atomicAdd(counter, __popcll(who));
    if (who) base = __shfl(base, __ffsll(who) - 1);
    return base + __popcll(who & ((1ull << lane) - 1));
  };
  const bool grouped = here && a != t;
  const int stored = before == 0 && own ? ~a : a;
  const bool starts3 = grouped && before % 3 == 0, starts2 = grouped && before % 2 == 0;
  const bool lone = here && a == t && before + behind == 0;
  const int at3 = append(starts3, lists + 1);
  const int at2 = append(starts2, lists);
  const int at1 = append(lone, lists + 2);
  // mixed: of the n tokens of the run the first 3 * threes go in threes
  const int n = before + behind + 1, threes = n % 3 == 1 ? (n - 4) / 3 : n / 3;
  if (grouped && n == 1) atomicOr(reinterpret_cast<unsigned *>(lists + 3), 0x80000000u);
  const bool mixed3 = grouped && n > 1 && before < 3 * threes && before % 3 == 0;
  const bool mixed2 = grouped && n > 1 && before >= 3 * threes && (before - 3 * threes) % 2 == 0;
  const int at_m3 = append(mixed3, lists + 3) & 0x7fffffff;
  const int at_m2 = append(mixed2, SimilarityLists::mixed_twos(lists, n_tok));
  if (mixed3) SimilarityLists::groups(lists, n_tok, 3)[n_tok - 1 - at_m3] = make_int4(stored, t, next[0], next[1]);
  if (mixed2) SimilarityLists::groups(lists, n_tok, 2)[n_tok - 1 - at_m2] = make_int4(stored, t, next[0], -1);
  if (starts3) SimilarityLists::groups(lists, n_tok, 3)[at3] = make_int4(stored, t, next[0], next[1]);
  if (starts2) SimilarityLists::groups(lists, n_tok, 2)[at2] = make_int4(stored, t, next[0], -1);
  if (lone) SimilarityLists::lone(lists, n_tok)[at1] = t;
}

// ---- one lane group: partner tok[0] and tokens tok[1..R] against all keys -------------------------
// The queries of a lane live in registers; with four of them at D = 128 (128 registers beside 64 of scores) the
// partner's goes to LDS behind the two K tiles, where the lane that wrote it reads it back for every MFMA.
template <int D, int R>
struct SimilarityLds {
  static constexpr bool PARTNER_IN_LDS = D == 128 && R == 3;
  static constexpr int PARTNER_OFF = 2 * RowBlock<D, SIM_BQ, SIM_BK>::TILE_BYTES;  // [wave][D / 16][lane] x 16 bytes
  static constexpr int RUN_OFF = PARTNER_OFF + (PARTNER_IN_LDS ? SIM_BQ * D * 2 : 0);  // the third level of sums:
  static constexpr int BYTES = RUN_OFF + (3 * R + 2) * SIM_BQ * 2 * 4;                 // float[3 R + 2][threads]
};

template <int D, int R>
struct SimilaritySums {
  float l[R + 1], sq[R + 1], dot[R + 1];  // row sum, sum of squares, sum of products with the partner (dot[0] unused)
};

template <int D, int R>
__device__ __forceinline__ SimilaritySums<D, R> similarity_pass(
    const RowBlock<D, SIM_BQ, SIM_BK> &rb, const u32x4 &Kres, const uint16_t *__restrict__ head_q,
    const int (&tok)[R + 1], const SimilarityDims &p) {
  using RB = RowBlock<D, SIM_BQ, SIM_BK>;
  constexpr int KB = RB::KB, DS = RB::DS, ROWB = RB::ROWB, TILE_BYTES = RB::TILE_BYTES, S = R + 1;
  // With two queries per lane there are registers for two score buffers: the MFMAs of a sub-tile then stand beside the
  // sums of the one before.
  constexpr bool PIPE = R == 1;
  static_assert(KB % 2 == 0, "the two score buffers alternate over the sub-tiles of a tile");
  // A query's reference is put SLACK above its largest logit so far and moves when a partial row sum against it reaches
  // SAFE, some 20 powers of two later; the arguments of the exponentials that matter, and so their rounding, stay as
  // small as those around a reference that lags by 10.  Error of the sums of rows whose first 64 keys lie 40 powers of two
  // below the rest (rms, D = 64 / 128) and time on activations with a positional component (30 heads of 2400 tokens, D =
  // 128): relative to the true maximum 2.4 / 2.6e-7; no slack and 2^40 3.6 / 3.4e-7, 119 us; no slack and 2^12 2.2 /
  // 2.3e-7, 154 us (references move in many steps); 2^10 and 2^12 2.1 / 2.3e-7, 119 us.
  constexpr float SLACK = 10.f;
  constexpr float SAFE = 0x1p12f;
  rb.issue_k_at(Kres, 0, 0);
  using L = SimilarityLds<D, R>;
  constexpr int FIRST = L::PARTNER_IN_LDS ? 1 : 0;  // first query in registers
  using Operand = typename RB::Operand;
  using Scores = f32x16[S];
  Operand q[S][DS];
  Operand *const partner_q = reinterpret_cast<Operand *>(rb.lds + L::PARTNER_OFF) + rb.wave * DS * 64 + rb.lane;
  if constexpr (L::PARTNER_IN_LDS) {
    rb.load_q(head_q + (size_t)tok[0] * D, q[0]);
#pragma unroll
    for (int d = 0; d < DS; ++d) partner_q[d * 64] = q[0][d];
  }
#pragma unroll
  for (int i = FIRST; i < S; ++i) rb.load_q(head_q + (size_t)tok[i] * D, q[i]);

  const int N = p.N, nbk = p.nbk;
  const float sc = p.scale_log2e;
  const bool ragged = (N % SIM_BK) != 0;
  // Three levels of sums - 16 logits, FLUSH tiles (32 such sums), all - so that no chain of fp32 additions is much
  // longer than the others: the rounding of a long chain is what the error of the result consists of.  The third
  // level is touched every FLUSH tiles and lives in LDS, each lane's own words.
  constexpr int FLUSH = 16;
  float *const run = reinterpret_cast<float *>(rb.lds + L::RUN_OFF) + rb.tid;
  auto run_l = [&](int i) -> float & { return run[i * RB::NT]; };
  auto run_sq = [&](int i) -> float & { return run[(S + i) * RB::NT]; };
  auto run_dot = [&](int i) -> float & { return run[(2 * S + i - 1) * RB::NT]; };  // i > 0
  SimilaritySums<D, R> mid;
  float m[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    m[i] = -INFINITY;
    run_l(i) = run_sq(i) = 0.f;
    if (i > 0) run_dot(i) = 0.f;
    mid.l[i] = mid.sq[i] = mid.dot[i] = 0.f;
  }
  // S of one 32-key sub-tile of the K tile at `tile`
  auto multiply = [&](const char *tile, int kb, Scores &s) {
    const char *const kbuf = tile + kb * 32 * ROWB;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[i][v] = 0.f;
#pragma unroll
    for (int d = 0; d < DS; ++d) {
      const Operand ka = *reinterpret_cast<const Operand *>(kbuf + (rb.k_addr0 ^ (d << 5)));
      if constexpr (L::PARTNER_IN_LDS) s[0] = Bf16::mfma(ka, partner_q[d * 64], s[0]);
#pragma unroll
      for (int i = FIRST; i < S; ++i) s[i] = Bf16::mfma(ka, q[i][d], s[i]);
    }
  };
  // keys >= N to -inf; the scale is applied up front, multiplier 1 from then on
  auto mask_tail = [&](Scores &s, int kb) {
    int limit = N - (nbk - 1) * SIM_BK - 32 * kb - 8 * rb.g;  // this lane's key offsets below `limit` exist
    asm volatile("" : "+v"(limit));                             // keeps the comparisons inside this branch
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[i][v] = 16 * (v >> 3) + (v & 7) < limit ? s[i][v] * sc : -INFINITY;
    return 1.0f;
  };
  auto fold = [&](const Scores &s, float sc_t) {
    SimilaritySums<D, R> part;
    auto sum = [&]() {
#pragma unroll
      for (int i = 0; i < S; ++i) part.l[i] = part.sq[i] = part.dot[i] = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float e[S];
#pragma unroll
        for (int i = 0; i < S; ++i) {
          e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][v], sc_t, -m[i]));
          part.l[i] += e[i];
          part.sq[i] = __builtin_fmaf(e[i], e[i], part.sq[i]);
          if (i > 0) part.dot[i] = __builtin_fmaf(e[i], e[0], part.dot[i]);
        }
      }
    };
    sum();
    bool bad = false;
#pragma unroll
    for (int i = 0; i < S; ++i) bad |= !(part.l[i] < SAFE);
    if (__any(bad)) {  // always on the first sub-tile, where the references are -inf
      float alpha[S];
#pragma unroll
      for (int i = 0; i < S; ++i) {
        float m_loc = sc_t >= 0.f ? -INFINITY : INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) m_loc = sc_t >= 0.f ? fmaxf(m_loc, s[i][v]) : fminf(m_loc, s[i][v]);
        // either half of the query's lanes out of range: both move
        const bool move = !(max_with_other_half(part.l[i] < SAFE ? 0.f : 1.f) < 0.5f);
        // finite also where every logit so far is -inf, so that their exponentials are 0
        const float m_new = move ? fmaxf(fmaxf(m[i], max_with_other_half(m_loc * sc_t) + SLACK), -FLT_MAX) : m[i];
        alpha[i] = move ? __builtin_amdgcn_exp2f(m[i] - m_new) : 1.f;  // 0 on the first sub-tile
        m[i] = m_new;
        run_l(i) *= alpha[i];
        mid.l[i] *= alpha[i];
        run_sq(i) *= alpha[i] * alpha[i];
        mid.sq[i] *= alpha[i] * alpha[i];
        if (i > 0) run_dot(i) *= alpha[i] * alpha[0];
        if (i > 0) mid.dot[i] *= alpha[i] * alpha[0];
      }
      sum();
    }
#pragma unroll
    for (int i = 0; i < S; ++i) {
      mid.l[i] += part.l[i];
      mid.sq[i] += part.sq[i];
      if (i > 0) mid.dot[i] += part.dot[i];
    }
  };
  auto flush = [&](int c) {
    if (c % FLUSH == FLUSH - 1 || c == nbk - 1) {
#pragma unroll
      for (int i = 0; i < S; ++i) {
        run_l(i) += mid.l[i];
        run_sq(i) += mid.sq[i];
        if (i > 0) run_dot(i) += mid.dot[i];
        mid.l[i] = mid.sq[i] = mid.dot[i] = 0.f;
      }
    }
  };
  Scores s[PIPE ? 2 : 1];
  for (int c = 0; c < nbk; ++c) {
    wait_vmem<0>();
    __syncthreads();  // tile c has landed for every wave; everyone is done with the other buffer
    if (c + 1 < nbk) rb.issue_k_at(Kres, c + 1, ((c + 1) & 1) * TILE_BYTES);
    const char *const tile = rb.ldsK + (c & 1) * TILE_BYTES;
    const bool tail = ragged && c == nbk - 1;
    if constexpr (PIPE) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        Scores &now = s[kb & 1], &before = s[(kb & 1) ^ 1];
        if (kb == 0 && c == 0) {
          multiply(tile, kb, now);
          continue;
        }
        float sc_t = sc;
        if (kb > 0 && tail) sc_t = mask_tail(before, kb - 1);
        multiply(tile, kb, now);
        fold(before, sc_t);
        if (kb == 0) flush(c - 1);
      }
    } else {
#pragma unroll 1
      for (int kb = 0; kb < KB; ++kb) {
        multiply(tile, kb, s[0]);
        fold(s[0], tail ? mask_tail(s[0], kb) : sc);
      }
      flush(c);
    }
  }
  if constexpr (PIPE) {
    fold(s[(KB - 1) & 1], ragged ? mask_tail(s[(KB - 1) & 1], KB - 1) : sc);
    flush(nbk - 1);
  }
  SimilaritySums<D, R> total;
  float w[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    total.l[i] = sum_with_other_half(run_l(i));
    w[i] = 1.0f / total.l[i];
    total.sq[i] = sum_with_other_half(run_sq(i)) * w[i] * w[i];
    total.dot[i] = i > 0 ? sum_with_other_half(run_dot(i)) * w[i] * w[0] : 0.f;
  }
  return total;
}

__device__ __forceinline__ void store_triple(float *__restrict__ head_triples, int t, float dot, float nt, float na) {
  float *const o = head_triples + (size_t)t * 3;
  o[0] = dot;
  o[1] = nt;
  o[2] = na;
}

// Position of a workgroup in the sequence of all units (units_per_head of each (batch, head)), cut into one
// contiguous range per XCD; false when it has none.
__device__ __forceinline__ bool similarity_unit(const SimilarityDims &p, int units_per_head, int &bh, int &r) {
  const int xcd = blockIdx.x % SIM_XCDS;
  const int slot = blockIdx.x / SIM_XCDS;
  const long long units = (long long)p.B * p.H * units_per_head;
  const long long lo = units * xcd / SIM_XCDS;
  const long long hi = units * (xcd + 1) / SIM_XCDS;
  if (slot >= hi - lo) return false;
  const int unit = (int)(lo + slot);
  r = unit % units_per_head;
  bh = unit / units_per_head;
  return true;
}

// Every token with its partner, without lists.
template <int D>
__device__ __forceinline__ void pair_similarity(char *lds, const uint16_t *__restrict__ gq,
                                                const uint16_t *__restrict__ gk, const int32_t *__restrict__ partner,
                                                float *__restrict__ triples, const SimilarityDims &p) {
  using RB = RowBlock<D, SIM_BQ, SIM_BK>;
  int bh, r;
  if (!similarity_unit(p, p.nbq, bh, r)) return;
  RB rb(lds);
  const size_t head_off = (size_t)bh * (size_t)p.N * D;
  const int tok_raw = r * SIM_BQ + rb.row_in_block();
  const int t = min(tok_raw, p.n_tok - 1);
  const int tok[2] = {similarity_partner(partner, t, p.N), t};
  const SimilaritySums<D, 1> sums =
      similarity_pass<D, 1>(rb, head_rsrc(gk + head_off, (uint32_t)p.N * RB::ROWB), gq + head_off, tok, p);
  if (tok_raw < p.n_tok && rb.g == 0)
    store_triple(triples + (size_t)bh * p.n_tok * 3, t, sums.dot[1], sums.sq[1], sums.sq[0]);
}

template <int D>
__global__ __launch_bounds__(SIM_BQ * 2, 2) void pair_similarity_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, const int32_t *__restrict__ partner,
    float *__restrict__ triples, const SimilarityDims p) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // SimilarityLds<D, 1>::BYTES
  pair_similarity<D>(lds, gq, gk, partner, triples, p);
}

// Unit `unit` of 128 lane groups of head bh: groups of the list at `groups` (step 1, or -1 from its far end), or lone tokens.
template <int D, int R>
__device__ __forceinline__ void grouped_similarity(char *lds, const uint16_t *__restrict__ gq,
                                                   const uint16_t *__restrict__ gk, int32_t *__restrict__ lists,
                                                   float *__restrict__ triples, const SimilarityDims &p,
                                                   const int4 *groups, int step, int n_groups, int n_lone, bool lone,
                                                   int bh, int unit) {
  using RB = RowBlock<D, SIM_BQ, SIM_BK>;
  RB rb(lds);
  const int at = unit * SIM_BQ + rb.row_in_block();
  int id[R + 1];
  bool own = false;
  if (lone) {  // R + 1 tokens that are their own partners per lane
#pragma unroll
    for (int i = 0; i <= R; ++i) {
      const int j = at * (R + 1) + i;
      id[i] = j < n_lone ? SimilarityLists::lone(lists, p.n_tok)[j] : -1;
    }
  } else if (at < n_groups) {
    const int4 g = groups[(long long)at * step];
    own = g.x < 0;
    id[0] = own ? ~g.x : g.x;
    id[1] = g.y;
    if constexpr (R > 1) id[2] = g.z;
    if constexpr (R > 2) id[3] = g.w;
  } else {
#pragma unroll
    for (int i = 0; i <= R; ++i) id[i] = -1;
  }
  int tok[R + 1];  // slots without a token repeat another one's work
#pragma unroll
  for (int i = 0; i <= R; ++i) tok[i] = id[i] >= 0 ? id[i] : max(id[0], 0);
  const size_t head_off = (size_t)bh * (size_t)p.N * D;
  const SimilaritySums<D, R> sums =
      similarity_pass<D, R>(rb, head_rsrc(gk + head_off, (uint32_t)p.N * RB::ROWB), gq + head_off, tok, p);
  if (rb.g != 0) return;
  float *const out = triples + (size_t)bh * p.n_tok * 3;
#pragma unroll
  for (int i = 0; i <= R; ++i) {
    if (id[i] < 0) continue;
    if (lone || (i == 0 && own))
      store_triple(out, id[i], sums.sq[i], sums.sq[i], sums.sq[i]);
    else if (i > 0)
      store_triple(out, id[i], sums.dot[i], sums.sq[i], sums.sq[0]);
  }
}

// Three tokens per group cost the fewest rows of logits, two waste fewer lanes on a short last group and are smaller
// units of work, tokens that share nothing are best off in pairs: the form with the fewest rows of logits on the CU that
// has the most to do is taken, two tokens before three (at D = 128 those keep the partner in LDS) and groups before pairs
// where that is the same.  `cus`: compute units of an XCD.  D = 128, ms in pairs / twos / threes (rows on the busiest CU):
//   24 heads of 21 x 30 x 52 tokens, five anchors   12.64 (48) /  9.84 (36) / 10.00 (36);  D = 64  9.39 / 7.41 / 7.23
//   5 heads of 21 x 45 x 80 tokens, three anchors   14.81 (24) / 11.71 (18) / 10.73 (16)
//   24 heads of 8 x 30 x 40 tokens, five anchors     1.23 (16) /  0.99 (12) /  1.00 (12), random partners 1.22 / 1.90 / 2.55
//   18 heads of 4 x 30 x 32 tokens, five anchors    0.196 (6)  / 0.203 (6)  / 0.176 (4)
template <int D>
__global__ __launch_bounds__(SIM_BQ * 2, 2) void grouped_similarity_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, const int32_t *__restrict__ partner,
    int32_t *__restrict__ lists, float *__restrict__ triples, const SimilarityDims p, int cus) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // SimilarityLds<D, 3>::BYTES
  const int n2 = lists[0], n3 = lists[1], n_lone = lists[2];
  auto rows = [&](int units_per_head, int queries) {
    const long long units = (long long)p.B * p.H * units_per_head;
    return ((units + SIM_XCDS - 1) / SIM_XCDS + cus - 1) / cus * queries;
  };
  auto grouped_rows = [&](int groups, int R) {
    const int lone = (n_lone + R) / (R + 1);
    return rows((groups + SIM_BQ - 1) / SIM_BQ + (lone + SIM_BQ - 1) / SIM_BQ, R + 1);
  };
  const long long rows3 = grouped_rows(n3, 3), rows2 = grouped_rows(n2, 2), rows1 = rows(p.nbq, 2);
  auto units = [](int n) { return (n + SIM_BQ - 1) / SIM_BQ; };
  // Mixed: units of four and of three rows of logits, evenly among each other (an XCD takes a range of them).
  const int m3 = lists[3], m2 = n_lone < p.n_tok ? *SimilarityLists::mixed_twos(lists, p.n_tok) : 0;
  const int u3 = m3 < 0 ? 0 : units(m3), u2 = units(m2), u1 = units((n_lone + 3) / 4);
  const int per_head = u3 + u2 + u1;
  const bool mixed = u3 > 0 && u2 > 0 && per_head <= p.nbq + 1 &&
                     rows(per_head, SIM_THREE_COST * (u3 + u1) + 30 * u2) * 10 <
                         SIM_MIXED_GAIN * per_head * min(rows1, min(rows2, rows3));
  if (!mixed && rows1 < min(rows2, rows3)) {
    pair_similarity<D>(lds, gq, gk, partner, triples, p);
    return;
  }
  const bool twos = !mixed && rows2 <= rows3;
  const int first = mixed ? u3 : twos ? units(n2) : units(n3);  // units of the first list, then of a second one
  const int second = mixed ? u2 : 0;
  int bh, r;
  if (!similarity_unit(p, first + second + (twos ? units((n_lone + 2) / 3) : u1), bh, r)) return;
  const bool lone = r >= first + second;
  const int before = lone ? first : (int)((long long)r * first / (first + second));  // units of the first list
  const bool of_second = !lone && (long long)(r + 1) * first / (first + second) == before;
  const int unit = lone ? r - first - second : of_second ? r - before : before;
  if (twos || of_second) {
    const int4 *const at = SimilarityLists::groups(lists, p.n_tok, 2) + (mixed ? p.n_tok - 1 : 0);
    grouped_similarity<D, 2>(lds, gq, gk, lists, triples, p, at, mixed ? -1 : 1, mixed ? m2 : n2, n_lone, lone, bh, unit);
  } else {
    const int4 *const at = SimilarityLists::groups(lists, p.n_tok, 3) + (mixed ? p.n_tok - 1 : 0);
    grouped_similarity<D, 3>(lds, gq, gk, lists, triples, p, at, mixed ? -1 : 1, mixed ? m3 : n3, n_lone, lone, bh, unit);
  }
}

// score[b*H + h] = mean over the n_tok / row_len spatial rows of the row's cosine.  A half wavefront adds the
// triples of one row at a time (lane x takes the columns x, x + 32, ...); the 32 rows in flight of a workgroup and
// then its half wavefronts are added in a fixed order.
constexpr int SIM_REDUCE_THREADS = 1024;
__global__ __launch_bounds__(SIM_REDUCE_THREADS) void similarity_reduce_kernel(const float *__restrict__ triples,
                                                                               float *__restrict__ score, int n_tok,
                                                                               int row_len) {
  constexpr int HALVES = SIM_REDUCE_THREADS / 32;
  __shared__ float part[HALVES];
  const int bh = blockIdx.x;
  const int n_rows = n_tok / row_len;
  const int half = threadIdx.x / 32, x0 = threadIdx.x % 32;
  const float *const base = triples + (size_t)bh * n_tok * 3;
  float acc = 0.f;
  for (int row0 = 0; row0 < n_rows; row0 += HALVES) {  // every lane takes part in the sums of every round
    const int row = row0 + half;
    float dot = 0.f, nt = 0.f, na = 0.f;
    if (row < n_rows)
      for (int x = x0; x < row_len; x += 32) {
        const float *const t = base + ((size_t)row * row_len + x) * 3;
        dot += t[0];
        nt += t[1];
        na += t[2];
      }
    dot = half_wave_sum(dot);
    nt = half_wave_sum(nt);
    na = half_wave_sum(na);
    if (row < n_rows) acc += dot / (sqrtf(nt) * sqrtf(na));
  }
  if (x0 == 0) part[half] = acc;
  __syncthreads();
  if (threadIdx.x < 64) {
    const float total = wave_sum(threadIdx.x < HALVES ? part[threadIdx.x] : 0.f);
    if (threadIdx.x == 0) score[bh] = total / (float)n_rows;
  }
}

}  // namespace calibatt_dev
