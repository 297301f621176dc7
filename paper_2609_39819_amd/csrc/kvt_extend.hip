// Extend attention over a paged KV cache, gfx950.
//
// The S_b new tokens of sequence b attend causally over the P_b reused
// positions plus themselves (prefix reuse in place of re-prefill, paper §1,
// §2.2).  Work decomposition, per workgroup:
//   * one kv-head g and 256 packed query rows (row r = token r/G, head
//     g*G + r%G): the G query heads that share a kv-head share every K/V
//     tile staged in LDS;
//   * 8 waves (two per SIMD), each owning 32 rows; the wave computes
//     S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (keys on the MFMA rows,
//     queries on the columns), so a query's scores sit in one lane pair
//     (l, l+32) and the row max / row sum need a single permlane32 swap;
//   * the probabilities leave the S^T accumulators already in the B-operand
//     layout of O^T += V^T P^T; the V^T operand comes straight from the
//     row-major V tile through ds_read_b64_tr_b16;
//   * fp32 online softmax in log2 units (scale*log2e folded into one FMA);
//   * K/V tiles of 64 keys (4 pages) are gathered through the block table
//     straight into a double-buffered LDS ring (global_load_lds_dwordx4);
//     every page contributes one contiguous run of 16*D elements per
//     kv-head, read with 16-byte coalesced loads; the next tile streams in
//     while the current one is computed.
// Positions past the end of the sequence and unused page slots are never
// multiplied in: their loads read the last real position instead (finite
// data) and their scores are replaced by -inf, so their weight is exactly 0.
#include "kvt_device.h"
#include "kvt_internal.h"

namespace kvt {
namespace {

using namespace dev;
constexpr int kThreads = kExtWaves * 64;

// One K or V tile of 64 keys in LDS: [key][D] bf16, the 16-byte chunks of
// each key row XOR-swizzled.  A ring slot is one object holding K then V, so
// every operand read of a slot is a per-lane offset plus an immediate; the
// two slots are distinct objects so the compiler can tell the page gather
// into one slot from the operand reads of the other.
template <int D>
struct HalfTile {
  __bf16 e[kExtKeysPerTile * D];
};
template <int D>
struct Slot {
  HalfTile<D>& k;
  HalfTile<D>& v;
};

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void extend_fwd_kernel(const ExtendArgs a) {
  constexpr int KT = kExtKeysPerTile;            // 64 keys per tile = 4 pages
  constexpr int CHUNKS = D / 8;                  // 16-byte chunks per key row
  constexpr int ROWB = D * 2;                    // bytes per key row in LDS
  constexpr int RPR = 1024 / ROWB;               // key rows per 1 KiB wave load
  constexpr int NREG = KT * ROWB / 1024 / kExtWaves;  // 1 KiB loads per wave per tensor
  constexpr int KSTEPS = D / 16;                 // MFMA k-steps of the score product
  constexpr int DT = D / 32;                     // 32-wide output column tiles
  constexpr bool kDirect = sizeof(T) == 2;       // bf16 storage: global -> LDS directly
  constexpr float kRescaleSlack = 8.0f;          // log2 headroom before O is rescaled
  constexpr int NB = kExtRowsPerWave / 32;       // 32-row MFMA blocks per wave
  __shared__ __attribute__((aligned(1024))) HalfTile<D> slot0[2];   // K, V
  __shared__ __attribute__((aligned(1024))) HalfTile<D> slot1[2];
  const Slot<D> tile0{slot0[0], slot0[1]}, tile1{slot1[0], slot1[1]};

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5;     // lane half
  const int l32 = lane & 31;

  // ---- which (sequence, kv-head, row tile, key split) this workgroup owns
  const int hkv = a.num_kv_heads;
  const int g = blockIdx.x % hkv;
  const int unit = blockIdx.x / hkv;
  const int si = find_seq(a.unit_begin, a.nseq, unit);
  const SeqDesc sd = a.seq[si];
  const int local = unit - a.unit_begin[si];
  // key range, splits and partial slots of this sequence's group
  const bool grp2 = si >= a.second;
  const int kbeg = grp2 ? a.kbeg2 : a.kbeg;
  const int kend = grp2 ? a.kend2 : a.kend;
  const int sets = grp2 ? a.nsplit2 : a.nsplit;   // partial sets, and key splits of every row tile but the last
  const int part_base = grp2 ? a.part_base2 : a.part_base;
  const int G = a.group;
  const int rows_seq = sd.suffix * G;
  const int ntile = (rows_seq + kExtTileRows - 1) / kExtTileRows;
  // longest (last) row tile first
  const int last = a.last[si];
  const bool last_tile = local < last;
  const int nsplit = last_tile ? last : sets;
  const int rest = last_tile ? local : local - last;
  const int rt = last_tile ? ntile - 1 : ntile - 2 - rest / sets;
  const int split = last_tile ? local : rest % sets;
  // partial slot of this unit, and how many of the sets after it hold no keys
  // for its rows (the last split marks them); one scalar across the tile loop
  const int slot_fill = (part_base + split) | (split == nsplit - 1 ? sets - nsplit : 0) << 16;
  const int r0 = rt * kExtTileRows;
  const int P = sd.prefix;
  const int L = min(P + sd.suffix, kend);      // positions that can be read
  const int nblk = (L + kBlock - 1) / kBlock;

  // keys this tile needs: from kbeg up to the last query's own position
  // (or kend); the range is split evenly over the key splits
  const int t_last = min(sd.suffix - 1, (r0 + kExtTileRows - 1) / G);
  const int kmax = min(P + t_last + 1, kend);
  const int ntiles_kv = (kmax + KT - 1) / KT;
  const int jlo = kbeg / KT;
  const int per_split = (ntiles_kv - jlo + nsplit - 1) / nsplit;
  const int j0 = jlo + split * per_split;
  const int j1 = min(ntiles_kv, j0 + per_split);
  const int lim_min = min(P + r0 / G, kend - 1);   // smallest last-visible key of the tile

  // ---- this lane's query rows: block b = rows kExtRowsPerWave*wave + 32*b + l32
  int lim[NB];
  bool row_valid[NB];
  int64_t qrow[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    int r = r0 + wave * kExtRowsPerWave + b * 32 + l32;
    row_valid[b] = r < rows_seq;
    if (!row_valid[b]) r = rows_seq - 1;
    const int t = r / G;
    const int h = g * G + (r - t * G);
    lim[b] = min(P + t, kend - 1);                    // last visible position
    qrow[b] = (int64_t)(sd.row_off + t) * a.num_q_heads + h;
  }
  bf16x8 qreg[NB][KSTEPS];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const T* qp = reinterpret_cast<const T*>(a.q) + qrow[b] * D;
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) qreg[b][kk] = __builtin_bit_cast(bf16x8, load8(qp + kk * 16 + hh * 8));
  }

  const T* kpool = reinterpret_cast<const T*>(a.k_pool);
  const T* vpool = reinterpret_cast<const T*>(a.v_pool);
  // the block table is read-only here: a constant-address-space view lets
  // wave-uniform page lookups become scalar loads
  const __attribute__((address_space(4))) int32_t* bt =
      (const __attribute__((address_space(4))) int32_t*)(a.block_table + (int64_t)sd.seq * a.max_blocks);
  const uint32_t nb_max = (uint32_t)min<int64_t>(a.num_blocks, 0x7fffffff) - 1u;

  // ---- gather geometry: wave w, load i covers key rows RPR*(w + 8i) ..
  // +RPR-1 of the tile, all inside one page.  Lane l lands at LDS byte
  // 16*l of that 1 KiB run, i.e. row RPR*(w + 8i) + l/CHUNKS, physical chunk
  // l%CHUNKS, so it fetches logical chunk (l%CHUNKS) ^ swizzle(row).
  constexpr uint32_t ROWM = D * sizeof(T) - 1;   // bytes of one stored key row, as a mask
  int lds_off[NREG], page_in_tile[NREG];
  uint32_t lane_off[NREG];                       // this lane's byte offset within its page run
#pragma unroll
  for (int i = 0; i < NREG; ++i) {
    const int run = wave + kExtWaves * i;
    const int keyrow = RPR * run + lane / CHUNKS;
    page_in_tile[i] = (RPR * run) / kBlock;
    lds_off[i] = run * 512;                                   // elements
    lane_off[i] = (uint32_t)(((keyrow & (kBlock - 1)) * D + (((lane % CHUNKS) ^ swz<D>(keyrow)) << 3)) * (int)sizeof(T));
  }
  // physical page ids of the pages a tile needs, as the block table has them
  // (wave-uniform scalar loads).  They are clamped into the pool where they
  // are used, a step later: clamped here, every wave waited for the loads in
  // the middle of its score product (128K reused + 2048 new tokens, 96/8
  // heads: 11.34 ms then, 11.20 ms now, same process)
  auto page_ids = [&](int jn, uint32_t (&ids)[NREG]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NREG; ++i) {
      const int page = __builtin_amdgcn_readfirstlane(min(jn * 4 + page_in_tile[i], nblk - 1));
      ids[i] = (uint32_t)bt[page];
    }
  };
  // A lane's piece lies at a byte offset within its page run; positions past
  // the end of the sequence take the offset of the last real position instead
  // (finite data whose weight is 0; lane_bytes, branch-free).
  // bf16 storage: global -> LDS by DMA.  The DMAs themselves (dma) carry no
  // branch either, so the score product can spread them between its matrix
  // instructions instead of every wave issuing all of them at once.
  const uint32_t tail = (uint32_t)((L - 1) & (kBlock - 1)) * (ROWM + 1);   // last real row of the last page
  auto lane_bytes = [&](int jn, uint32_t (&lb)[NREG]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NREG; ++i) {
      // byte of the page's last real row (not formed from the rows left after
      // the page: in long contexts those are more than 2^32 bytes)
      const uint32_t last = jn * 4 + page_in_tile[i] >= nblk - 1 ? tail : (kBlock - 1) * (ROWM + 1);
      lb[i] = min(lane_off[i], last | (lane_off[i] & ROWM));
    }
  };
  auto dma = [&](uint32_t id, uint32_t lb, int i, const Slot<D>& dst) __attribute__((always_inline)) {
    const int64_t base = (((int64_t)min(id, nb_max) * hkv + g) << 4) * D;
    const char* ks = reinterpret_cast<const char*>(kpool + base) + lb;
    const char* vs = reinterpret_cast<const char*>(vpool + base) + lb;
    lds_bf16* kd = (lds_bf16*)dst.k.e + lds_off[i];
    lds_bf16* vd = (lds_bf16*)dst.v.e + lds_off[i];
    __builtin_amdgcn_global_load_lds((const void*)ks, (__attribute__((address_space(3))) void*)kd, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)vs, (__attribute__((address_space(3))) void*)vd, 16, 0, 0);
  };
  // fp32 storage: a tile's pieces are loaded into registers as they are
  // stored (issue_staged, before the score product of the tile ahead of it)
  // and rounded to bf16 and put into LDS after that tile's value product
  // (stash), so the loads have a whole tile's compute to land in.  Rounded
  // and stored right after the loads, every tile waited for HBM first: 8192
  // reused + 512 new tokens, 32/8 heads of 64, append + extend + merge, 67.5 us
  // per pass then, 58.2 us now; 16384 + 8192 tokens, 32/8 heads of 128,
  // 3.06 ms and 2.66 ms.
  f32x4 stK[NREG][2], stV[NREG][2];
  auto issue_staged = [&](const uint32_t (&ids)[NREG], const uint32_t (&lb)[NREG]) __attribute__((always_inline)) {
    if constexpr (!kDirect) {
#pragma unroll
      for (int i = 0; i < NREG; ++i) {
        const int64_t base = (((int64_t)min(ids[i], nb_max) * hkv + g) << 4) * D;
        const char* ks = reinterpret_cast<const char*>(kpool + base) + lb[i];
        const char* vs = reinterpret_cast<const char*>(vpool + base) + lb[i];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          stK[i][p] = *reinterpret_cast<const f32x4*>(ks + 16 * p);
          stV[i][p] = *reinterpret_cast<const f32x4*>(vs + 16 * p);
        }
      }
    }
  };
  auto stash = [&](const Slot<D>& dst) __attribute__((always_inline)) {
    if constexpr (!kDirect) {
#pragma unroll
      for (int i = 0; i < NREG; ++i) {
        *reinterpret_cast<u32x4*>(dst.k.e + lds_off[i] + lane * 8) = round8(stK[i][0], stK[i][1]);
        *reinterpret_cast<u32x4*>(dst.v.e + lds_off[i] + lane * 8) = round8(stV[i][0], stV[i][1]);
      }
    }
  };

  f32x16 o[NB][DT];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[b][dt] = (f32x16){};
  // m_ref: reference max of scale*log2e*score (trails the true max by less
  // than the slack); l_run: this lane's share of sum 2^(s*c - m_ref)
  float m_ref[NB], l_run[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) m_ref[b] = -INFINITY, l_run[b] = 0.f;
  const float c = a.scale_log2;
  const int g16 = (lane >> 4) & 1;
  const int rsel = (lane & 15) >> 2;

  // lane-constant LDS element offsets of the MFMA operand reads; the 32-key
  // half and 16-key group parts are compile-time constants
  int koff[KSTEPS], voff[DT][2];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) koff[kk] = l32 * D + (((2 * kk + hh) ^ swz<D>(l32)) << 3);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2) {
      const int key = 8 * r2 + 4 * hh + rsel;          // key within a 16-key group
      const int dcol = dt * 32 + g16 * 16 + 4 * (lane & 3);
      voff[dt][r2] = key * D + (((dcol >> 3) ^ swz<D>(key)) << 3) + (dcol & 7);
    }
  // ---- S^T = K Q^T of one tile: two independent 32-key accumulator chains
  // per 32-row block, each K fragment read from LDS feeding NB blocks.  With
  // bf16 storage it also issues the gather of the next tile into `fill`
  // (page ids, lane offsets lb), one DMA after each of score steps 1 .. 2*NREG.
  auto qk = [&](const Slot<D>& tl, f32x16 (&s)[NB][2], const uint32_t (&ids)[NREG], const uint32_t (&lb)[NREG],
                const Slot<D>& fill) __attribute__((always_inline)) {
    const __bf16* ks = tl.k.e;
    if constexpr (kDirect) {
#pragma unroll
      for (int i = 0; i < NREG; ++i) dma(ids[i], lb[i], i, fill);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) s[b][0] = s[b][1] = (f32x16){};
    bf16x8 kf[KSTEPS][2];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      kf[kk][0] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ks + koff[kk]));
      kf[kk][1] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ks + koff[kk] + 32 * D));
    }
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        s[b][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk][0], qreg[b][kk], s[b][0], 0, 0, 0);
        s[b][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk][1], qreg[b][kk], s[b][1], 0, 0, 0);
      }
    }
    // K fragments read ahead of the products that use them: two steps'
    // worth first, then each pair of products followed by the next pair of
    // reads and (after steps 1 .. 2*NREG) one gather DMA
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int kk = 0; kk < KSTEPS - 2; ++kk) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * NB, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      if (kDirect && kk >= 1 && kk <= 2 * NREG) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4 * NB, 0);
  };
  // ---- between tiles: causal mask of tile j (only tiles reaching past the
  // tile's first query), row max, and the reference-max update.  The
  // reference only moves when a tile max passes it by more than the slack;
  // O and l are then rescaled (rare after the first tiles).
  // Element e of half h of a lane's scores is key j*KT + 4*hh + koff(h, e)
  // with koff(h, e) = 32h + 8(e/4) + e%4 in 0..59: the masks compare that
  // constant against one per-lane threshold, so no key index is formed.
  auto settle = [&](int j, f32x16 (&s)[NB][2]) __attribute__((always_inline)) {
    if (j * KT + KT - 1 > lim_min) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int thr = lim[b] - j * KT - 4 * hh;        // keys past lim: koff > thr
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (half * 32 + 8 * (e >> 2) + (e & 3) > thr) s[b][half][e] = -INFINITY;
      }
    }
    if (j * KT < kbeg) {   // first tile of a range that starts inside it
      const int thr = kbeg - j * KT - 4 * hh;          // keys before kbeg: koff < thr
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (half * 32 + 8 * (e >> 2) + (e & 3) < thr) s[b][half][e] = -INFINITY;
    }
    float alpha[NB];
    bool moved = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float mx = -INFINITY;
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[b][half][e]);
      const float mxc = pair_max(mx) * c;
      const float m_new = (mxc > m_ref[b] + kRescaleSlack) ? mxc : m_ref[b];
      // 1 when unchanged, 0 when leaving -inf; kept at 1 while the row has
      // seen no visible key (a key split can lie wholly past a row's limit)
      alpha[b] = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_ref[b] - m_new);
      m_ref[b] = m_new;
      l_run[b] *= alpha[b];
      moved = moved || alpha[b] != 1.0f;
    }
    if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[b][dt] *= alpha[b];
    }
  };
  // ---- probabilities of a settled tile: P^T as the B operand of the value
  // product (key group kg = 16 keys); the row sum adds the bf16 values the
  // value product uses
  auto probs = [&](f32x16 (&s)[NB][2], bf16x8 (&pb)[NB][4]) __attribute__((always_inline)) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float m_use = (m_ref[b] == -INFINITY) ? 0.f : m_ref[b];
      float rs = 0.f;
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) {
        const int half = kg >> 1, b0 = (kg & 1) * 8;
        u32x4 wv;
#pragma unroll
        for (int q2 = 0; q2 < 4; ++q2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][half][b0 + 2 * q2], c, -m_use));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][half][b0 + 2 * q2 + 1], c, -m_use));
          const bf16x2 pp = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
          rs = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, rs, false);
          wv[q2] = __builtin_bit_cast(unsigned, pp);
        }
        pb[b][kg] = __builtin_bit_cast(bf16x8, wv);
      }
      l_run[b] += rs;
    }
  };
  // ---- O^T += V^T P^T; V^T comes from the row-major tile by transposed
  // reads, each fragment feeding NB MFMAs
  auto pv = [&](const Slot<D>& tl, const bf16x8 (&pb)[NB][4]) __attribute__((always_inline)) {
    const lds_bf16* vl = (const lds_bf16*)tl.v.e;
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vl + voff[dt][0] + kg * 16 * D));
        const bf16x4 v2 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(vl + voff[dt][1] + kg * 16 * D));
        const bf16x8 vf = __builtin_shufflevector(v1, v2, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          o[b][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pb[b][kg], o[b][dt], 0, 0, 0);
      }
    }
  };

  // ---- main loop.  Step t computes tile t (scores, settle, probabilities,
  // value product) and, inside the score product, gathers tile t+1 into the
  // other slot (its page ids were fetched a step earlier; past the last
  // tile the gather still reads clamped, in-bounds pages into a slot no one
  // reads).  The wait + barrier at the end publishes tile t+1 and frees the
  // slot of tile t for the gather of tile t+2.
  const int n = j1 - j0;
  uint32_t ids[NREG], lb[NREG];
  page_ids(j0, ids);
  if (n > 0) {
    lane_bytes(j0, lb);
    if constexpr (kDirect) {
#pragma unroll
      for (int i = 0; i < NREG; ++i) dma(ids[i], lb[i], i, tile0);
    } else {
      issue_staged(ids, lb);
      stash(tile0);
    }
  }
  page_ids(j0 + 1, ids);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  __syncthreads();
  f32x16 s_cur[NB][2];
  bf16x8 pb[NB][4];
  auto step = [&](int t, const Slot<D>& cur, const Slot<D>& fill) __attribute__((always_inline)) {
    lane_bytes(j0 + t + 1, lb);
    if (t + 1 < n) issue_staged(ids, lb);
    qk(cur, s_cur, ids, lb, fill);
    page_ids(j0 + t + 2, ids);
    settle(j0 + t, s_cur);
    probs(s_cur, pb);
    pv(cur, pb);
    if (!kDirect && t + 1 < n) stash(fill);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);   // see the loop below
  };
  if (r0 + wave * kExtRowsPerWave >= rows_seq) {
    // A wave past the sequence's last row only takes its part in the gather:
    // no products or softmax for padding (67 new tokens x 4 heads over 30011
    // keys, a full row tile and one of 12 rows: 69.1 us per pass with them,
    // 61.0 without; ragged batch of 8 contexts, 755 and 725 us).
    auto gather = [&](int t, const Slot<D>& fill) __attribute__((always_inline)) {
      lane_bytes(j0 + t + 1, lb);
      if constexpr (kDirect) {
#pragma unroll
        for (int i = 0; i < NREG; ++i) dma(ids[i], lb[i], i, fill);
      } else if (t + 1 < n) {
        issue_staged(ids, lb);
        stash(fill);
      }
      page_ids(j0 + t + 2, ids);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
    };
    for (int t = 0; t < n; t += 2) {
      gather(t, tile1);
      if (t + 1 >= n) break;
      gather(t + 1, tile0);
    }
    return;
  }
  // Two steps per pass without a branch between them, the scheduler held at
  // the end of each: the compiler places the last products and the barrier
  // differently with every other change of the kernel, and some of those
  // placements cost 2 to 6 % (128K reused + 2048 new tokens: 11.28 ms this
  // way, 11.30 the best of the others, 11.46 to 11.95 with the loop above
  // added and left to the compiler; same process).
  int t = 0;
  for (; t + 2 <= n; t += 2) {
    step(t, tile0, tile1);
    step(t + 1, tile1, tile0);
  }
  if (t < n) step(t, tile0, tile1);

  // ---- epilogue
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float l_tot = pair_sum(l_run[b]);
    if (!row_valid[b]) continue;
    if (a.direct) {
      const float inv = 1.0f / l_tot;
      T* op = reinterpret_cast<T*>(a.out) + qrow[b] * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = dt * 32 + 8 * i + 4 * hh;
          store4(op + d, o[b][dt][4 * i] * inv, o[b][dt][4 * i + 1] * inv, o[b][dt][4 * i + 2] * inv,
                 o[b][dt][4 * i + 3] * inv);
        }
      if (a.lse != nullptr && hh == 0) a.lse[qrow[b]] = (m_ref[b] + __builtin_log2f(l_tot)) * kLn2;
    } else {
      const int slot = slot_fill & 0xffff, fill = slot_fill >> 16;
      const int64_t set_rows = (int64_t)a.total_rows * a.num_q_heads;
      const int64_t prow = slot * set_rows + qrow[b];
      float* op = a.part_o + prow * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = dt * 32 + 8 * i + 4 * hh;
          store4(op + d, o[b][dt][4 * i], o[b][dt][4 * i + 1], o[b][dt][4 * i + 2], o[b][dt][4 * i + 3]);
        }
      if (hh == 0) {
        a.part_ml[prow * 2] = m_ref[b];
        a.part_ml[prow * 2 + 1] = l_tot;
        for (int s = 1; s <= fill; ++s) {
          a.part_ml[(prow + s * set_rows) * 2] = -INFINITY;
          a.part_ml[(prow + s * set_rows) * 2 + 1] = -1.f;   // its O is not written
        }
      }
    }
  }
}

// Merge the per-split partial results of each row (fixed split order):
//   m* = max_s m_s,  w_s = 2^(m_s - m*),  out = sum_s w_s O_s / sum_s w_s l_s.
// A set that holds no keys for a row has m = -inf there.  Where the plan gives
// some row tiles fewer splits (gaps), the sets that those do not have were
// never written: they are marked by l = -1 and left out.  Every other set is
// multiplied by its weight, be it 0, so an infinity or a NaN among the values
// gives the unsplit call's.
// One thread per 16 columns of a row: four 16-byte loads per split in flight,
// and each split's (m, l) read once per 16 columns.
template <typename T, int D>
__global__ __launch_bounds__(256) void extend_combine_kernel(const CombineArgs a) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (row, 16-column group)
  constexpr int Q16 = D / 16;
  if (idx >= a.rows * Q16) return;
  const int64_t row = idx / Q16;
  const int c16 = (int)(idx - row * Q16) * 16;
  float mstar = -INFINITY;
  for (int s = 0; s < a.nsplit; ++s) mstar = fmaxf(mstar, a.part_ml[(s * a.rows + row) * 2]);
  float lsum = 0.f;
  f32x4 acc[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int s = 0; s < a.nsplit; ++s) {
    const int64_t pr = s * a.rows + row;
    const float m = a.part_ml[pr * 2];
    const float w = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mstar);
    const float l = a.part_ml[pr * 2 + 1];
    lsum += w * l;
    const f32x4* src = reinterpret_cast<const f32x4*>(a.part_o + pr * D + c16);
    f32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = src[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (a.gaps && l < 0.f) v[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
      acc[k] += w * v[k];
    }
  }
  const float inv = 1.0f / lsum;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    store4(reinterpret_cast<T*>(a.out) + row * D + c16 + 4 * k, acc[k][0] * inv, acc[k][1] * inv, acc[k][2] * inv,
           acc[k][3] * inv);
  if (a.lse != nullptr && c16 == 0) a.lse[row] = (mstar + __builtin_log2f(lsum)) * kLn2;
}

// The same merge for calls with few rows (a decoding step, a short message),
// which is bound by memory round trips instead of bytes.  One thread per 4
// columns, so a row's D/4 lanes also load the (m, l) pairs of its splits, one
// each, turn them into weights there and share those through LDS; the O
// pieces of kCombineAhead splits are loaded before that, all in flight at once.
// Kernel time with this kernel [with the one above]: 96 rows x 16 splits
// 4.2 us [11.1], 2144 x 16 5.6 [11.3], 16384 x 4 of 64 columns 5.0 [5.8];
// 16384 x 4 of 128 columns 8.1 [7.5], 49152 x 4 19.4 [18.0].  It takes the calls
// with fewer than 2^16 (row, 16-column group) pairs, where the kernel above has
// less than one workgroup per CU, and with five and more splits (fp32: four),
// whose round trips add up there, those with fewer than 2^17.  Time of a call
// with this kernel less that with the one above, bf16 of 128 columns, at 2, 4, 8
// and 16 splits: 6144 rows +0.2, -0.3, -1.1, -2.6 us; 9216 rows +1.1, +0.6,
// -0.8, -2.1; 12288 rows +1.1, +0.5, -0.1, -0.4; 16368 rows +1.1, +0.7, +0.5,
// +0.8; fp32 of 64 columns at 2 and 4: 16320 rows +0.5, -0.4; 24576 rows +0.4,
// -0.5.
constexpr int kCombineAhead = 16;
constexpr int64_t kCombineFewBelow = 1 << 16;   // (row, 16-column group) pairs; twice that from
template <typename T>                           // this many splits on
constexpr int kCombineManySplits = sizeof(T) == 4 ? 4 : 5;

template <typename T, int D, bool GAPS>
__global__ __launch_bounds__(256) void extend_combine_few_kernel(const CombineArgs a) {
  constexpr int Q4 = D / 4, ROWS = 256 / Q4;     // lanes per row, rows per workgroup
  __shared__ float wts[ROWS][kMaxPartials + 1];
  const int lr = threadIdx.x / Q4, q = threadIdx.x % Q4;
  const int64_t row0 = (int64_t)blockIdx.x * ROWS + lr;
  const bool live = row0 < a.rows;
  const int64_t row = live ? row0 : a.rows - 1;
  const float* po = a.part_o + row * D + q * 4;
  const f32x2* pml = reinterpret_cast<const f32x2*>(a.part_ml) + row;
  const int64_t ostep = a.rows * D;
  f32x4 v[kCombineAhead];
#pragma unroll
  for (int i = 0; i < kCombineAhead; ++i)
    if (i < a.nsplit) v[i] = *reinterpret_cast<const f32x4*>(po + i * ostep);
  constexpr int PER = (kMaxPartials + Q4 - 1) / Q4;   // splits per lane
  float m[PER], l[PER];
  float mstar = -INFINITY;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int s = q + k * Q4;
    m[k] = -INFINITY, l[k] = 0.f;
    if (s < a.nsplit) {
      const f32x2 e = pml[s * a.rows];
      m[k] = e[0], l[k] = e[1];
    }
    mstar = fmaxf(mstar, m[k]);
  }
#pragma unroll
  for (int d = Q4 / 2; d > 0; d >>= 1) mstar = fmaxf(mstar, __shfl_xor(mstar, d));
  float lsum = 0.f;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int s = q + k * Q4;
    const float w = (m[k] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m[k] - mstar);
    lsum += w * l[k];
    if (s < a.nsplit) wts[lr][s] = GAPS && l[k] < 0.f ? -1.f : w;   // -1: not written
  }
#pragma unroll
  for (int d = Q4 / 2; d > 0; d >>= 1) lsum += __shfl_xor(lsum, d);
  __syncthreads();
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kCombineAhead; ++i)
      if (s0 + i < a.nsplit) {
        const float w = wts[lr][s0 + i];
        acc += w * (GAPS && w < 0.f ? (f32x4){0.f, 0.f, 0.f, 0.f} : v[i]);
      }
  };
  add(0);
  for (int s0 = kCombineAhead; s0 < a.nsplit; s0 += kCombineAhead) {
#pragma unroll
    for (int i = 0; i < kCombineAhead; ++i)
      if (s0 + i < a.nsplit) v[i] = *reinterpret_cast<const f32x4*>(po + (s0 + i) * ostep);
    add(s0);
  }
  if (!live) return;
  const float inv = 1.0f / lsum;
  store4(reinterpret_cast<T*>(a.out) + row * D + q * 4, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  if (a.lse != nullptr && q == 0) a.lse[row] = (mstar + __builtin_log2f(lsum)) * kLn2;
}

}  // namespace

hipError_t launch_extend(const ExtendArgs& a, int dtype, int head_dim, int grid, hipStream_t stream) {
  dim3 g(grid), b(kThreads);
  if (dtype == 0 && head_dim == 128) hipLaunchKernelGGL((extend_fwd_kernel<__bf16, 128>), g, b, 0, stream, a);
  else if (dtype == 0 && head_dim == 64) hipLaunchKernelGGL((extend_fwd_kernel<__bf16, 64>), g, b, 0, stream, a);
  else if (dtype == 1 && head_dim == 128) hipLaunchKernelGGL((extend_fwd_kernel<float, 128>), g, b, 0, stream, a);
  else hipLaunchKernelGGL((extend_fwd_kernel<float, 64>), g, b, 0, stream, a);
  return hipGetLastError();
}

template <typename T, int D>
void launch_combine_as(const CombineArgs& a, hipStream_t stream) {
  const int64_t n16 = a.rows * (D / 16);
  if (n16 < (a.nsplit < kCombineManySplits<T> ? kCombineFewBelow : 2 * kCombineFewBelow)) {
    const int64_t per = 256 / (D / 4);
    const dim3 grid((unsigned)((a.rows + per - 1) / per)), block(256);
    if (a.gaps) hipLaunchKernelGGL((extend_combine_few_kernel<T, D, true>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((extend_combine_few_kernel<T, D, false>), grid, block, 0, stream, a);
  } else {
    hipLaunchKernelGGL((extend_combine_kernel<T, D>), dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, stream, a);
  }
}

hipError_t launch_combine(const CombineArgs& a, int dtype, int head_dim, hipStream_t stream) {
  if (dtype == 0 && head_dim == 128) launch_combine_as<__bf16, 128>(a, stream);
  else if (dtype == 0 && head_dim == 64) launch_combine_as<__bf16, 64>(a, stream);
  else if (dtype == 1 && head_dim == 128) launch_combine_as<float, 128>(a, stream);
  else launch_combine_as<float, 64>(a, stream);
  return hipGetLastError();
}

}  // namespace kvt
