// Block energy of an attention map without materialising it (paper, Section
// 3.2, Eq. 5): E[r][c] = mean over the queries of block r of the softmax mass
// they put on the keys of block c.  gfx950 (MI355X), bf16 in, fp32 out.
//
// One workgroup per (batch, head, query block), two passes over all key tiles
// with the QK^T engine of the attention kernels (RowBlock::scores; a lane owns
// one query and half of the tile's keys):
//   pass 1  running row max and row sum (online softmax statistics);
//   pass 2  p = exp2(s - max) / sum per entry, summed over the lane's keys,
//           then over the wave's 32 queries with a fixed butterfly, one fp32
//           partial per (wave, key block) in LDS; at the end the partials of
//           the workgroup's waves are added in wave order and divided by the
//           number of rows the block has.
// No V, so both LDS tile buffers hold K: tile c+1 streams in while tile c is
// multiplied, one barrier per tile.  Work units are placed like those of the
// anchor kernel (contiguous ranges per XCD) since all query blocks of a head
// walk the same K tiles in step.  Every addition order is fixed: the result is
// the same bits on every run.
#pragma once
#include "attn_kernel_2wg.h"

namespace calibatt_dev {

struct EnergyDims {
  int B, H, N, nbq, nbk;
  float scale_log2e;
};

constexpr int ENERGY_XCDS = 8;

template <int D, int BQ, int BK>
struct EnergyLds {
  using RB = RowBlock<D, BQ, BK>;
  static constexpr int PART_OFF = 2 * RB::TILE_BYTES;  // float[NW][nbk] partial sums behind the two K buffers
  static __host__ __device__ constexpr long long bytes(int nbk) { return PART_OFF + (long long)RB::NW * nbk * 4; }
};

template <int D, int BQ, int BK>
__global__ __launch_bounds__(BQ * 2, (BQ >= 128 ? 2 : 1)) void block_energy_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, float *__restrict__ gE, const EnergyDims p) {
  using RB = RowBlock<D, BQ, BK>;
  constexpr int NT = RB::NT, NW = RB::NW, KB = RB::KB, ROWB = RB::ROWB, TILE_BYTES = RB::TILE_BYTES;

  extern __shared__ __attribute__((aligned(1024))) char lds[];  // EnergyLds::bytes(nbk)

  const int xcd = blockIdx.x % ENERGY_XCDS;
  const int slot = blockIdx.x / ENERGY_XCDS;
  const long long units = (long long)p.B * p.H * p.nbq;
  const long long lo = units * xcd / ENERGY_XCDS;
  const long long hi = units * (xcd + 1) / ENERGY_XCDS;
  if (slot >= hi - lo) return;
  const int unit = (int)(lo + slot);
  const int r = unit % p.nbq;
  const int bh = unit / p.nbq;  // b * H + h

  RB rb(lds);
  const int tid = rb.tid;
  const int N = p.N;
  const size_t head_off = (size_t)bh * (size_t)N * D;
  const u32x4 Kres = head_rsrc(gk + head_off, (uint32_t)N * ROWB);
  float *const part = reinterpret_cast<float *>(lds + EnergyLds<D, BQ, BK>::PART_OFF);
  const int rows_valid = min(BQ, N - r * BQ);

  rb.template issue_k_at<true>(Kres, 0, 0);
  const bool row_valid = rb.row_in_block() < rows_valid;
  rb.begin(gq + head_off + (size_t)(r * BQ + (row_valid ? rb.row_in_block() : 0)) * D);
  const float sc = p.scale_log2e;
  const bool ragged = (N % BK) != 0;

  float m_run = -INFINITY, l_run = 0.f, weight = 0.f;
  // Tiles of both passes form one sequence t = pass * nbk + c; tile t sits in buffer t & 1.
  const int n_steps = 2 * p.nbk;
  for (int t = 0; t < n_steps; ++t) {
    const bool second = t >= p.nbk;
    const int c = second ? t - p.nbk : t;
    wait_vmem<0>();
    __syncthreads();  // tile t has landed for every wave; everyone is done with the other buffer
    if (t + 1 < n_steps) rb.template issue_k_at<true>(Kres, c + 1 < p.nbk ? c + 1 : 0, ((t + 1) & 1) * TILE_BYTES);
    f32x16 s[KB];
    rb.scores((t & 1) * TILE_BYTES, s);
    // Work on the raw products with the scale folded into the exponent's FMA; only the ragged last
    // tile is scaled up front so that its keys >= N can sit at -inf (multiplier 1 from then on).
    float sc_t = sc;
    if (ragged && c == p.nbk - 1) {
      int limit = N - c * BK - 8 * rb.g;  // this lane's key offsets below `limit` exist
      asm volatile("" : "+v"(limit));      // keeps the comparisons (and their 64 masks) inside this branch
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          s[kb][v] = 32 * kb + 16 * (v >> 3) + (v & 7) < limit ? s[kb][v] * sc : -INFINITY;
      sc_t = 1.0f;
    }
    if (!second) {
      // largest scaled logit of the tile: the largest product, or the smallest under a negative scale
      float m_loc;
      if (sc_t >= 0.f) {
        m_loc = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) m_loc = fmaxf(m_loc, s[kb][v]);
      } else {
        m_loc = INFINITY;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) m_loc = fminf(m_loc, s[kb][v]);
      }
      const float m_new = fmaxf(m_run, max_with_other_half(m_loc * sc_t));
      float psum = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) psum += __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][v], sc_t, -m_new));
      l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_new) + psum;
      m_run = m_new;
      if (c == p.nbk - 1) weight = row_valid ? 1.0f / sum_with_other_half(l_run) : 0.f;
    } else {
      float e = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) e += __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][v], sc_t, -m_run));
      e = wave_sum(e * weight);
      if (rb.lane == 0) part[rb.wave * p.nbk + c] = e;
    }
  }
  __syncthreads();
  const float inv_rows = 1.0f / (float)rows_valid;
  float *const out = gE + ((size_t)bh * p.nbq + r) * (size_t)p.nbk;
  for (int c = tid; c < p.nbk; c += NT) {
    float e = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) e += part[w * p.nbk + c];
    out[c] = e * inv_rows;
  }
}

// The same energies in ONE pass over the key tiles, for callers that bring a
// workspace.  While the online-softmax statistics of a row are still running,
// the mass it puts on key block c is only known relative to the running
// maximum of that moment; its logarithm, t[c][row] = m + log2(sum over the
// block's keys of 2^(s - m)), needs no reference.  A workgroup keeps these
// nbk x QW values in its slice of the workspace and, once the row's
// log-sum-exp L is known, reads its own values back:
// E[r][c] = mean over the rows of 2^(t[c][row] - L[row]).  Every lane reads
// only what it wrote itself.  Half the matrix work of the two-pass kernel;
// 2 x nbk x BQ x 4 bytes of extra traffic per query block.
//
// The reference of the exponentials only has to keep them in range, it need
// not be the maximum: a tile is first summed against the reference as it
// stands, and only if some lane's sum leaves the safe range (always on the
// first tile, where the reference is -inf) do the 32 rows that a wavefront
// holds together look for the tile's maximum, move their references and sum
// again.  The sums stay below 2^100 per tile, so the row sum cannot overflow.
//
// All forms give the same bits: the same additions in the same order in a
// lane, the same 32 rows that move their references together and whose masses
// are added as one partial.  Which one runs, on how many workgroups, is a
// matter of speed alone.
//
// Persistent workgroups, no counters: workgroup i serves XCD i mod xcds and
// takes every (workgroups of that XCD)-th unit of the XCD's contiguous range;
// all units cost the same.  The workspace slice belongs to the workgroup, not
// to the unit.
struct EnergyOnePassDims {
  EnergyDims e;
  int n_wg;     // workgroups launched
  int xcds;     // 8, or 1 when fewer than 8 workgroups run
  int n_group;  // units per head: ceil(nbq / BLOCKS)
};

constexpr float ENERGY_SAFE = 0x1p100f;  // largest sum of one tile against the present reference

// This workgroup's units: lo + slot, lo + slot + step, ... below hi.
struct EnergyUnits {
  long long first, hi;
  int step;
  __device__ __forceinline__ explicit EnergyUnits(const EnergyOnePassDims &pp) {
    const int xcd = blockIdx.x % pp.xcds;
    const long long units = (long long)pp.e.B * pp.e.H * pp.n_group;
    first = units * xcd / pp.xcds + blockIdx.x / pp.xcds;
    hi = units * (xcd + 1) / pp.xcds;
    step = (pp.n_wg - xcd + pp.xcds - 1) / pp.xcds;
  }
};

// partial[group][c], one per 32 rows, to the energies of the workgroup's query blocks
template <int BQ, int BLOCKS, int NT>
__device__ __forceinline__ void store_energies(const float *partial, float *__restrict__ gE, long long bh, int r0,
                                               const EnergyDims &p, int tid) {
#pragma unroll
  for (int j = 0; j < BLOCKS; ++j) {
    const int r = r0 + j;
    if (r >= p.nbq) break;
    const float inv_rows = 1.0f / (float)min(BQ, p.N - r * BQ);
    float *const out = gE + ((size_t)bh * p.nbq + r) * (size_t)p.nbk;
    for (int c = tid; c < p.nbk; c += NT) {
      float e = 0.f;
#pragma unroll
      for (int w = 0; w < BQ / 32; ++w) e += partial[(j * (BQ / 32) + w) * p.nbk + c];
      out[c] = e * inv_rows;
    }
  }
}

// Narrow form: a wavefront owns 32 queries, QW of them (one query block, or two of 64) make a workgroup.
template <int D, int BQ, int BK, int QW>
struct EnergyOnePass {
  static constexpr int NW = QW / 32;      // wavefronts per workgroup
  static constexpr int BLOCKS = QW / BQ;  // query blocks per workgroup
  static constexpr int QUERIES = QW;
  using RB = RowBlock<D, QW, BK>;
  static constexpr int PART_OFF = 2 * RB::TILE_BYTES;  // float[NW][nbk] partial sums behind the two K buffers
  static __host__ __device__ constexpr long long bytes(int nbk) { return PART_OFF + (long long)NW * nbk * 4; }
};

// Two wavefronts per SIMD in the bounds also where a workgroup has only two: with the whole register file to itself a
// wavefront's scores go to accumulation registers and are copied out before they are used.
template <int D, int BQ, int BK, int QW>
__global__ __launch_bounds__(QW * 2, 2) void block_energy_onepass_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, float *__restrict__ gE,
    float *__restrict__ workspace, const EnergyOnePassDims pp) {
  using L = EnergyOnePass<D, BQ, BK, QW>;
  using RB = typename L::RB;
  constexpr int NT = RB::NT, KB = RB::KB, ROWB = RB::ROWB, TILE_BYTES = RB::TILE_BYTES;
  const EnergyDims &p = pp.e;

  extern __shared__ __attribute__((aligned(1024))) char lds[];  // L::bytes(nbk)

  RB rb(lds);
  const int N = p.N;
  float *const part = reinterpret_cast<float *>(lds + L::PART_OFF);
  float *const mine = workspace + (size_t)blockIdx.x * p.nbk * QW + rb.row_in_block();  // + c * QW
  const float sc = p.scale_log2e;
  const bool ragged = (N % BK) != 0;

  const EnergyUnits units(pp);
  for (long long unit = units.first; unit < units.hi; unit += units.step) {
    const int r0 = (int)(unit % pp.n_group) * L::BLOCKS;
    const long long bh = unit / pp.n_group;  // b * H + h
    const size_t head_off = (size_t)bh * (size_t)N * D;
    const u32x4 Kres = head_rsrc(gk + head_off, (uint32_t)N * ROWB);
    const int row = r0 * BQ + rb.row_in_block();
    const bool row_valid = row < N;

    // both K buffers are free: every wave is behind the barrier that followed the last tile of the previous unit
    rb.template issue_k_at<true>(Kres, 0, 0);
    // a lane without a row of its own repeats the first row of its block
    rb.begin(gq + head_off + (size_t)(row_valid ? row : min(row / BQ * BQ, N - 1)) * D);

    float m_run = -INFINITY, l_run = 0.f, t_prev = 0.f;
    for (int c = 0; c < p.nbk; ++c) {
      wait_vmem<0>();
      __syncthreads();  // tile c has landed for every wave; everyone is done with the other buffer
      // the value of the previous tile goes out here, a whole tile ahead of the next wait for memory
      if (c > 0 && ((c - 1) & 1) == rb.g) mine[(size_t)(c - 1) * QW] = t_prev;
      if (c + 1 < p.nbk) rb.template issue_k_at<true>(Kres, c + 1, ((c + 1) & 1) * TILE_BYTES);
      f32x16 s[KB];
      rb.scores((c & 1) * TILE_BYTES, s);
      float sc_t = sc;
      if (ragged && c == p.nbk - 1) {  // keys >= N sit at -inf; the tile is scaled up front, multiplier 1 from then on
        int limit = N - c * BK - 8 * rb.g;  // this lane's key offsets below `limit` exist
        asm volatile("" : "+v"(limit));      // keeps the comparisons (and their 64 masks) inside this branch
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            s[kb][v] = 32 * kb + 16 * (v >> 3) + (v & 7) < limit ? s[kb][v] * sc : -INFINITY;
        sc_t = 1.0f;
      }
      float psum = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) psum += __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][v], sc_t, -m_run));
      if (__any(!(psum < ENERGY_SAFE))) {
        float m_loc;
        if (sc_t >= 0.f) {
          m_loc = -INFINITY;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) m_loc = fmaxf(m_loc, s[kb][v]);
        } else {
          m_loc = INFINITY;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) m_loc = fminf(m_loc, s[kb][v]);
        }
        const float m_new = fmaxf(m_run, max_with_other_half(m_loc * sc_t));
        psum = 0.f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) psum += __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][v], sc_t, -m_new));
        l_run *= __builtin_amdgcn_exp2f(m_run - m_new);  // 0 on the first tile
        m_run = m_new;
      }
      l_run += psum;
      // log2 of the row's mass on this block (-inf when it underflowed: the block then counts as 0)
      t_prev = m_run + __builtin_amdgcn_logf(sum_with_other_half(psum));
    }
    if (((p.nbk - 1) & 1) == rb.g) mine[(size_t)(p.nbk - 1) * QW] = t_prev;
    const float lse2 = m_run + __builtin_amdgcn_logf(sum_with_other_half(l_run));
    wait_vmem<0>();
    __syncthreads();  // K buffers free for the next unit; `part` of the previous unit fully consumed
    // this lane's own values back (blocks c = 2 j + g), 16 loads in flight at a time; each half of
    // the wave sums its 32 rows
    for (int c0 = 0; c0 < p.nbk; c0 += 32) {
      float t[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = c0 + 2 * j + rb.g;
        t[j] = c < p.nbk ? __hip_atomic_load(mine + (size_t)c * QW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                         : -INFINITY;  // read at L2, where the stores went
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = c0 + 2 * j + rb.g;
        const float e = half_wave_sum(row_valid ? __builtin_amdgcn_exp2f(t[j] - lse2) : 0.f);
        if (rb.l32 == 0 && c < p.nbk) part[rb.wave * p.nbk + c] = e;
      }
    }
    __syncthreads();
    store_energies<BQ, L::BLOCKS, NT>(part, gE, bh, r0, p, rb.tid);
  }
}

// Overlapped form: a wavefront owns one or two panels of 32 queries, four of them make a workgroup.
//
// What bounds the pass: the vector ALU (FMA, exponential and addition per logit) beside the matrix cores; a 32 x 32
// sub-tile is 8 MFMAs and 48 vector instructions per wavefront.  So the wavefront's stream is one step per 32 keys in
// which the MFMAs of step j and the vector instructions of step j - 1 are independent (two score buffers); with two
// panels a K operand read from LDS feeds two MFMAs, and a K tile loaded into LDS serves 256 queries.  The order inside a
// step is left to the compiler.  With one panel a lone workgroup on its CU is faster than the narrow form's (522 units of
// 33325 keys, D = 128: 852 -> 780 us), two on a CU, which overlap one another anyway, are slower (480 units of 2560 keys
// 47.5 -> 50.3 us).
//
// The scores of a tile are gone when its sum turns out to be out of range; they are then multiplied again from K in
// memory.  That is rare, as the references start at the maximum of the first tile, which is multiplied once more for it.
template <int D, int BQ, int BK, int PANELS>
struct EnergyPanels {
  static constexpr int NW = 4, QUERIES = NW * 32 * PANELS, BLOCKS = QUERIES / BQ;
  using RB = RowBlock<D, NW * 32, BK>;
  // float[NW * PANELS][nbk] partial sums over the second K buffer, which the next unit's loads reach behind a barrier
  static constexpr int PART_OFF = RB::TILE_BYTES;
  static __host__ __device__ constexpr long long bytes(int nbk) {
    const long long part = (long long)NW * PANELS * nbk * 4;
    return PART_OFF + (part > RB::TILE_BYTES ? part : RB::TILE_BYTES);
  }
};

template <int D, int BQ, int BK, int PANELS>
__global__ __launch_bounds__(256, 2) void block_energy_panels_kernel(
    const uint16_t *__restrict__ gq, const uint16_t *__restrict__ gk, float *__restrict__ gE,
    float *__restrict__ workspace, const EnergyOnePassDims pp) {
  using L = EnergyPanels<D, BQ, BK, PANELS>;
  using RB = typename L::RB;
  constexpr int NT = RB::NT, KB = RB::KB, DS = RB::DS, ROWB = RB::ROWB, QW = L::QUERIES;
  constexpr int TILE_BYTES = RB::TILE_BYTES, LAST = PANELS - 1;
  static_assert(KB % 2 == 0, "the two score buffers alternate over the steps of a tile");
  using Operand = typename RB::Operand;
  using Scores = f32x16[PANELS];
  const EnergyDims &p = pp.e;

  extern __shared__ __attribute__((aligned(1024))) char lds[];  // L::bytes(nbk)

  RB rb(lds);
  const int N = p.N, nbk = p.nbk;
  float *const part = reinterpret_cast<float *>(lds + L::PART_OFF);
  // this lane's values, + c * QW: row l32 of panel g of every block c, or of the only panel and every second block
  const int half = PANELS == 1 ? 0 : rb.g;
  float *const mine = workspace + (size_t)blockIdx.x * nbk * QW + rb.wave * 32 * PANELS + 32 * half + rb.l32;
  const float sc = p.scale_log2e;
  const bool ragged = (N % BK) != 0;

  const EnergyUnits units(pp);
  for (long long unit = units.first; unit < units.hi; unit += units.step) {
    const int r0 = (int)(unit % pp.n_group) * L::BLOCKS;
    const long long bh = unit / pp.n_group;  // b * H + h
    const size_t head_off = (size_t)bh * (size_t)N * D;
    const uint16_t *const head_k = gk + head_off;
    const u32x4 Kres = head_rsrc(head_k, (uint32_t)N * ROWB);
    const int row0 = r0 * BQ + rb.wave * 32 * PANELS + rb.l32;  // this lane's row of panel 0; of panel 1: + 32

    // both K buffers are free: every wave is behind the barrier that followed the last tile of the previous unit
    rb.template issue_k_at<true>(Kres, 0, 0);
    Operand q[PANELS][DS];
#pragma unroll
    for (int i = 0; i < PANELS; ++i) {  // a lane without a row of its own repeats the first row of its block
      const int row = row0 + 32 * i;
      rb.load_q(gq + head_off + (size_t)(row < N ? row : min(row / BQ * BQ, N - 1)) * D, q[i]);
    }

    // S of one 32-key sub-tile against the K operands of its DS slabs
    auto products = [&](const Operand (&ka)[DS], Scores &dst) {
#pragma unroll
      for (int i = 0; i < PANELS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) dst[i][v] = 0.f;
#pragma unroll
      for (int d = 0; d < DS; ++d)
#pragma unroll
        for (int i = 0; i < PANELS; ++i) dst[i] = Bf16::mfma(ka[d], q[i][d], dst[i]);
    };
    auto multiply = [&](uint32_t buf_off, int kb, Scores &dst) {  // kb of the tile at buf_off
      const char *const kbuf = rb.ldsK + buf_off + kb * 32 * ROWB;
      Operand ka[DS];
#pragma unroll
      for (int d = 0; d < DS; ++d) ka[d] = *reinterpret_cast<const Operand *>(kbuf + (rb.k_addr0 ^ (d << 5)));
      products(ka, dst);
    };
    auto multiply_again = [&](int c, int kb, Scores &dst) {  // the same from memory
      const int key = c * BK + kb * 32 + ((rb.l32 & 0x13) | ((rb.l32 & 4) << 1) | ((rb.l32 & 8) >> 1));
      const uint16_t *const krow = head_k + (size_t)min(key, N - 1) * D + 8 * rb.g;
      Operand ka[DS];
#pragma unroll
      for (int d = 0; d < DS; ++d) ka[d] = *reinterpret_cast<const Operand *>(krow + 16 * d);
      products(ka, dst);
    };
    // keys >= N of the ragged last tile to -inf, the scale applied up front (returns the multiplier left: 1)
    auto mask_tail = [&](Scores &src, int kb) {
      int limit = N - (nbk - 1) * BK - 32 * kb - 8 * rb.g;  // this lane's key offsets below `limit` exist
      asm volatile("" : "+v"(limit));                        // keeps the comparisons inside this branch
      // Twelve wait states between the last MFMA and a read of its result: the compiler's own wait falls short on the
      // path that enters this branch at once (the build checks the distance).
#pragma unroll
      for (int i = 0; i < PANELS; ++i) asm volatile("s_nop 11" : "+v"(src[i]));
#pragma unroll
      for (int i = 0; i < PANELS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) src[i][v] = 16 * (v >> 3) + (v & 7) < limit ? src[i][v] * sc : -INFINITY;
      return 1.0f;
    };
    // largest scaled logit so far: the largest product, or the smallest under a negative scale
    float m_run[PANELS], l_run[PANELS], psum[PANELS], m_loc[PANELS];
    auto fold_max = [&](const Scores &src, float sc_t) {
#pragma unroll
      for (int i = 0; i < PANELS; ++i) {
        float m = sc_t >= 0.f ? -INFINITY : INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) m = sc_t >= 0.f ? fmaxf(m, src[i][v]) : fminf(m, src[i][v]);
        m_loc[i] = fmaxf(m_loc[i], m * sc_t);
      }
    };
    // this lane's share of the mass of one sub-tile relative to the present reference
    auto exp_sum = [&](const Scores &src, float sc_t) {
#pragma unroll
      for (int i = 0; i < PANELS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) psum[i] += __builtin_amdgcn_exp2f(__builtin_fmaf(src[i][v], sc_t, -m_run[i]));
      // keeps the sums in their step: the compiler would move those of a whole tile behind its last MFMA
      asm volatile("" : "+v"(psum[0]), "+v"(psum[LAST]));
    };
    // tile c is summed: its logarithm (-inf when the mass underflowed: the block then counts as 0) to the workspace
    auto finish_tile = [&](int c, Scores &tmp) {
      bool moves[PANELS];
#pragma unroll
      for (int i = 0; i < PANELS; ++i) moves[i] = __any(!(psum[i] < ENERGY_SAFE));
      if (moves[0] || moves[LAST]) {
        const bool tail = ragged && c == nbk - 1;
        float sum_before[PANELS];
#pragma unroll
        for (int i = 0; i < PANELS; ++i) {
          sum_before[i] = psum[i];
          m_loc[i] = -INFINITY;
          psum[i] = 0.f;
        }
#pragma unroll 1
        for (int kb = 0; kb < KB; ++kb) {
          multiply_again(c, kb, tmp);
          fold_max(tmp, tail ? mask_tail(tmp, kb) : sc);
        }
#pragma unroll
        for (int i = 0; i < PANELS; ++i) {
          const float m_new = moves[i] ? fmaxf(m_run[i], max_with_other_half(m_loc[i])) : m_run[i];
          l_run[i] *= moves[i] ? __builtin_amdgcn_exp2f(m_run[i] - m_new) : 1.f;
          m_run[i] = m_new;
        }
#pragma unroll 1
        for (int kb = 0; kb < KB; ++kb) {
          multiply_again(c, kb, tmp);
          exp_sum(tmp, tail ? mask_tail(tmp, kb) : sc);
        }
#pragma unroll
        for (int i = 0; i < PANELS; ++i) psum[i] = moves[i] ? psum[i] : sum_before[i];
      }
      float t[PANELS];
#pragma unroll
      for (int i = 0; i < PANELS; ++i) {
        t[i] = m_run[i] + __builtin_amdgcn_logf(sum_with_other_half(psum[i]));
        l_run[i] += psum[i];
        psum[i] = 0.f;
      }
      if (PANELS == 2 || (c & 1) == rb.g) mine[(size_t)c * QW] = half ? t[LAST] : t[0];
    };

    Scores s[2];
#pragma unroll
    for (int i = 0; i < PANELS; ++i) {
      l_run[i] = psum[i] = 0.f;
      m_loc[i] = -INFINITY;
    }
    for (int c = 0; c < nbk; ++c) {
      wait_vmem<0>();
      __syncthreads();  // tile c has landed for every wave; everyone is done with the other buffer
      if (c + 1 < nbk) rb.template issue_k_at<true>(Kres, c + 1, ((c + 1) & 1) * TILE_BYTES);
      const uint32_t buf = (c & 1) * TILE_BYTES;
      const bool tail = ragged && c == nbk - 1;
      if (c == 0) {
#pragma unroll 1
        for (int kb = 0; kb < KB; ++kb) {
          multiply(buf, kb, s[0]);
          fold_max(s[0], tail ? mask_tail(s[0], kb) : sc);
        }
#pragma unroll
        for (int i = 0; i < PANELS; ++i) m_run[i] = max_with_other_half(m_loc[i]);
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        Scores &now = s[kb & 1], &before = s[(kb & 1) ^ 1];
        if (kb == 0 && c == 0) {
          multiply(buf, kb, now);
          continue;
        }
        float sc_t = sc;
        if (kb > 0 && tail) sc_t = mask_tail(before, kb - 1);
        multiply(buf, kb, now);
        exp_sum(before, sc_t);
        if (kb == 0) finish_tile(c - 1, before);
      }
    }
    {
      Scores &last = s[(KB - 1) & 1];
      exp_sum(last, ragged ? mask_tail(last, KB - 1) : sc);
      finish_tile(nbk - 1, last);
    }
    float lse2[PANELS];
#pragma unroll
    for (int i = 0; i < PANELS; ++i) lse2[i] = m_run[i] + __builtin_amdgcn_logf(sum_with_other_half(l_run[i]));
    wait_vmem<0>();
    __syncthreads();  // every wave is done with the K buffers
    // this lane's own values back, 16 loads in flight at a time, read at L2, where the stores went; each half of the
    // wave sums the 32 rows of its panel, or those of the only one for every second block
    const float my_lse = half ? lse2[LAST] : lse2[0];
    const bool my_row = row0 + 32 * half < N;
    constexpr int STEP = PANELS == 1 ? 2 : 1;  // blocks c that the wave takes per load
    for (int c0 = 0; c0 < nbk; c0 += 16 * STEP) {
      float t[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = c0 + STEP * j + (STEP == 2 ? rb.g : 0);
        t[j] = c < nbk ? __hip_atomic_load(mine + (size_t)c * QW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                       : -INFINITY;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = c0 + STEP * j + (STEP == 2 ? rb.g : 0);
        const float e = half_wave_sum(my_row ? __builtin_amdgcn_exp2f(t[j] - my_lse) : 0.f);
        if (rb.l32 == 0 && c < nbk) part[(rb.wave * PANELS + half) * nbk + c] = e;
      }
    }
    __syncthreads();
    store_energies<BQ, L::BLOCKS, NT>(part, gE, bh, r0, p, rb.tid);
  }
}

}  // namespace calibatt_dev
