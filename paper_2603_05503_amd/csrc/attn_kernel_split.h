// The interleaved forward (attn_kernel_il.h) with its rows cut along the keys.
//
// A row of key blocks is a chain: its sub-tiles go through one workgroup one after the other, 0.97 us per 64 keys at
// D = 128 where the workgroup has its CU to itself (a wavefront's issue of some 280 instructions; windows of four
// sub-tiles, loaded two stages earlier, change nothing) and more where two share it.  A call of few rows, or of a few long
// ones, lasts as long as the longest chain while most CUs idle.  Here the host cuts every row into parts of about equal
// length (split_plan.cpp), one workgroup takes one part, leaves its sums in a workspace, and the one that finds itself
// last adds them up.  Rows that are not cut go the same way: one workgroup each, the longest first, by the hardware's
// dispatcher instead of the counters.
// Measured (us, whole rows -> by plan; uniform masks, density 0.35 where not given): one head of 8 190 tokens 68 -> 31, four
// 77 -> 70, twelve 184 -> 161; two heads of 16 380 at 0.25 98 -> 84, one with all blocks kept 246 -> 137; twenty of 5 070,
// 64-query blocks, D = 64, 162 -> 70.  Adding up costs 0.6 us per part of a row, 67 KB each at D = 128.
#pragma once
#include "attn_kernel_il.h"

namespace calibatt_dev {

// Record of a part, three int4: {row id or -1, first entry in the row, entries, first entry in col_idx},
// {first and last interval word of the row, first block in fan_dst that repeats the row, number of these},
// {part | parts of the row << 16, batch index, slot of part 0 in the workspace, cut row}.
constexpr int PART_RECORD = 3;

struct FwdSplit {
  int32_t *arrivals;  // [n_rows] parts of a cut row that have left their sums
  float *workspace;   // [n_slots] of IlPart::FLOATS
};

template <int D, int BQ, int BK, typename T>
struct IlPart : IlRow<D, BQ, BK, T> {
  using Base = IlRow<D, BQ, BK, T>;
  using Base::A_O;
  using Base::DB;
  using Base::NT;
  using Base::V_S;
  using Base::Base;
  // A part leaves its sums as they lie in the registers: O^T in pieces of four accumulators, piece i of thread t at
  // [i][t] (1 KB per wavefront and store), then every thread's reference and row sum.
  static constexpr int PIECES = 4 * DB;
  static constexpr int FLOATS = (4 * PIECES + 2) * NT;

  // parts: of the row, in scalar registers
  __device__ __forceinline__ void store_part(float *parts, int part) const {
    const uint32_t off = (uint32_t)part * (FLOATS * 4) + this->tid * 16;
    static_unroll<PIECES>([&](auto i) { agent_store_acc_b128<A_O + 4 * i>(parts, off + i * NT * 16); });
    float *const ml = parts + (size_t)part * FLOATS + 4 * PIECES * NT + 2 * this->tid;
    agent_store_f32x2(ml, f32x2{this->m_run, this->l_run});
  }

  // The row's sums from those of its n_parts parts, in the order of the keys whichever workgroup does it: relative to
  // the largest reference M, O = sum_s 2^(m_s - M) O_s and likewise the row sums.  Half of a part's pieces is on its
  // way, into the registers of the score buffers, while the other half is added.  weights: LDS, a pair per part and
  // thread.
  __device__ __forceinline__ void merge_parts(const float *parts, int n_parts, f32x2 *weights) {
    const float *const ml = parts + 4 * PIECES * NT + 2 * this->tid;  // references and row sums of this thread
    float m = -FLT_MAX;
#pragma unroll 4
    for (int s = 0; s < n_parts; ++s) {
      const f32x2 x = agent_load_f32x2(ml + (size_t)s * FLOATS);
      weights[s * NT + this->tid] = x;
      m = fmaxf(m, x[0]);
    }
    float l = 0.f;
    for (int s = 0; s < n_parts; ++s) {
      f32x2 x = weights[s * NT + this->tid];
      x[0] = __builtin_amdgcn_exp2f(x[0] - m);
      weights[s * NT + this->tid] = x;
      l += x[0] * x[1];
    }
    this->m_run = m;
    this->l_run = l;
    static_unroll<16 * DB>([&](auto i) { acc_write<A_O + i>(0.f); });
    constexpr int HALF = PIECES / 2;
    auto request = [&](int s, auto half) {
      const uint32_t off = (uint32_t)min(s, n_parts - 1) * (FLOATS * 4) + this->tid * 16;
      static_unroll<HALF>([&](auto i) {
        constexpr int piece = half * HALF + i;
        agent_load_named_b128<V_S + 4 * piece>(parts, off + piece * NT * 16);
      });
    };
    auto add = [&](float w, auto half) {
      wait_vmem<HALF>();
      static_unroll<4 * HALF>([&](auto e) {
        constexpr int at = 4 * half * HALF + e;
        acc_write<A_O + at>(named_fma<V_S + at>(w, acc_read<A_O + at>()));
      });
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};
    request(0, first);
    request(0, second);
    for (int s = 0; s < n_parts; ++s) {
      const float w = weights[s * NT + this->tid][0];
      add(w, first);
      request(s + 1, first);  // behind the last part: the last again, not used
      add(w, second);
      request(s + 1, second);
    }
    wait_vmem<0>();
  }

};

template <int D, int BQ, int BK, bool IV, typename T>
__global__ __launch_bounds__(BQ * 2, (BQ >= 128 ? 2 : 1)) __attribute__((amdgpu_num_vgpr(IL_VGPRS))) void sparse_attn_fwd_split_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, const uint16_t *__restrict__ gv,
    uint16_t *__restrict__ gout, const int4 *__restrict__ parts, const int32_t *__restrict__ col_idx,
    const uint32_t *__restrict__ iv, const int32_t *__restrict__ fan_dst, const int32_t *__restrict__ head_map,
    float *__restrict__ lse, const FwdDims p, const FwdSplit split) {
  using Row = IlPart<D, BQ, BK, T>;
  constexpr int NT = Row::NT, ROWB = Row::ROWB, LDS_BYTES = Row::LDS_BYTES, COLS = il_iv_cols(BQ);
  il_claim_registers();

  // LDS as in sparse_attn_fwd_il_kernel
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int *const cols = reinterpret_cast<int *>(lds + LDS_BYTES + 64);
  volatile int *const mailbox = reinterpret_cast<volatile int *>(lds + LDS_BYTES);
  int rec = blockIdx.x * PART_RECORD;
  const int4 what = parts[rec];
  const int id = what.x, first = what.y, n_tiles = what.z, cbeg = what.w;
  if (id < 0) return;  // the lists of the XCDs differ in length
  Row rb(lds, (uint32_t)p.in.n * 2);
  const int tid = rb.tid;
  const int N = p.N;
  const int h = id / p.nbq;
  const int r = id - h * p.nbq;
  const int ht = head_map ? head_map[h] : h;
  if ((unsigned)ht >= (unsigned)p.H) return;
  const int b = parts[rec + 2].y;
  const size_t head_off = (size_t)b * p.in.b + (size_t)ht * p.in.h;
  const uint32_t head_bytes = (uint32_t)(N - 1) * rb.kv_row_bytes + ROWB;
  const u32x4 Kres = head_rsrc(gk + head_off, head_bytes);
  const u32x4 Vres = head_rsrc(gv + head_off, head_bytes);
  // IV: entries [from, from + COLS) of the part are expanded from the row's runs into LDS
  int chunk_lo = first;
  auto expand_runs = [&](int from) {
    chunk_lo = first + from;
    const int4 lists = parts[rec + 1];
    for (int i = lists.x + tid; i < lists.y; i += NT) {  // the word behind them only terminates the row
      const uint32_t w = iv[i], w_next = iv[i + 1];
      const int start = (int)(w & 0xffffu), before = (int)(w >> 16), len = (int)(w_next >> 16) - before;
      const int j0 = max(0, chunk_lo - before), j1 = min(len, min(chunk_lo + COLS, first + n_tiles) - before);
      for (int j = j0; j < j1; ++j) cols[before + j - chunk_lo] = start + j;
    }
    __syncthreads();
  };
  if constexpr (IV) expand_runs(0);
  auto col_at = [&](int entry) { return IV ? cols[first + entry - chunk_lo] : col_idx[cbeg + entry]; };
  const int qrow = min(r * BQ + rb.row_in_block(), N - 1);
  il_run_row<BK, IV, COLS>(rb, gq + head_off + (size_t)qrow * p.in.n, Kres, Vres, N, n_tiles, p.scale_log2e, col_at,
                           expand_runs);
  __syncthreads();  // every wave is done with the tile windows
  asm volatile("" : "+s"(rec));  // read the rest of the record only here: scalar registers are scarce in the stream
  const int4 where = parts[rec + 2];
  const int part = where.x & 0xffff, n_parts = __builtin_amdgcn_readfirstlane(where.x >> 16);
  if (n_parts > 1) {
    // Leave the part's sums; the workgroup that is the last to do so goes on with those of the whole row.  The parts'
    // workgroups may sit behind different L2s, so the sums are stored and loaded at agent scope: they are past the L2
    // when the wait in front of the barrier ends, and the part is counted behind that barrier.  (With plain stores and a
    // release fence in front of the count, every part pays a write-back of its XCD's L2, one at a time: 720 rows in
    // 2 088 parts take 161 us instead of 101.)
    const uint64_t at = reinterpret_cast<uint64_t>(split.workspace + (size_t)where.z * Row::FLOATS);
    float *const row_parts = reinterpret_cast<float *>(  // in scalar registers, for the loads of the merge
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(at >> 32)) << 32 |
        (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)at));
    rb.store_part(row_parts, part);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    if (tid == 0) {
      int32_t *const arrived = split.arrivals + where.w;
      const int before = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (before == n_parts - 1) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *mailbox = before;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(*mailbox) != n_parts - 1) return;
    asm volatile("" : : : "memory");
    rb.merge_parts(row_parts, n_parts, reinterpret_cast<f32x2 *>(lds));
    __syncthreads();
  }
  const int4 lists = parts[rec + 1];
  il_store_row(rb, lds, p, where.y, ht, r, fan_dst + lists.z, lists.w, gout, lse);
}

}  // namespace calibatt_dev
