// Flash attention of a chunk's queries over a stream's keys on gfx950 MFMA.
//
// o = softmax(q K^T / sqrt(d)) V per (stream, head) over keys [0, kv_len),
// every key visible (the chunk attends to its whole cache and to itself; the
// block-causal structure across chunks is what the cache holds).  Keys come
// either from frame pages through the stream's page table (self-attention)
// or from one contiguous per-stream block (text cross-attention); both store
// keys [H][T][d] and values transposed [H][d][T].
//
// Work item = (stream, head, 256-query tile): a 512-thread workgroup, eight
// waves of 32 query rows.  Key tiles of 64 are staged in LDS (keys row-major,
// values d-major, 16-byte chunks XOR-swizzled across banks) in four slots, by
// direct loads three tiles ahead.  Per wave and tile:
//   S^T = K Q^T   on v_mfma_f32_16x16x32_bf16 (K from LDS, Q held in VGPRs),
//   online softmax in fp32 with exp2 (log2(e)/sqrt(d) folded into one FMA),
//   O^T += V^T P^T on the same MFMA, P taken straight from the S registers,
// the two waves of a SIMD half a tile apart (attn_range).
// Computing the transposed products puts one query row in each lane column,
// so the row max needs two cross-lane exchanges and no LDS round trip.  The
// keys of a tile are stored in LDS in the order kappa16 below, which makes
// the S values a lane holds for PV step s exactly the 8 keys that lane
// supplies to the P operand: P needs no shuffle and each V^T operand is one
// 16-byte LDS read.  Fragment reads are issued four ahead of the MFMAs that
// consume them.
//
// When the items are so few that one workgroup per item would leave more than
// a quarter of the CUs idle, and it ends sooner, each item keeps the first part of
// its key range and the idle workgroups share the remaining parts; the pieces leave
// partial results (unnormalised O, running max and denominator in fp32) that a second
// kernel merges.  A last round of items that leaves as many idle is cut the same
// way after the full rounds (plan_attention).  Calls of few queries over few keys
// take workgroups of 32 queries that split the keys between their waves
// (attn_small_kernel).
#include <math.h>
#include <string.h>

#include <type_traits>

#include "launch.h"

namespace ardit {

namespace {

constexpr int BQ = 256;        // queries per work item
constexpr int BKV = 64;        // keys per tile
constexpr int NTHR = 512;      // threads per workgroup
constexpr int LDS_AHEAD = 4;   // fragment reads in flight ahead of the MFMAs
constexpr int NSLOT = 4;       // key and value tiles in LDS

// Key order of a 64-key tile for 16x16x32 MFMAs: row r of 16-key block kb
// holds physical key kappa(kb, r) = 32 (kb/2) + 8 (r/4) + 4 (kb%2) + r%4, so
// the S^T values a lane holds for blocks 2s and 2s+1 are exactly keys
// 32 s + 8 g .. 32 s + 8 g + 7 (g = lane / 16): the P operand of PV step s.
__device__ __forceinline__ int kappa16(int kb, int r) {
  return 32 * (kb >> 1) + 8 * (r >> 2) + 4 * (kb & 1) + (r & 3);
}
// 16-byte chunk c of LDS row r sits at chunk c ^ swz(r): 16 consecutive rows
// then cover every bank for a fixed c.  Rows of 256 bytes (keys, d = 128) use
// r % 16, rows of 128 bytes (keys d = 64, values) (r / 2) % 8.
template <int ROWB>
__device__ __forceinline__ int swz(int r) { return ROWB == 256 ? (r & 15) : ((r >> 1) & 7); }

// Keys of one 64-key tile: [j0, j0 + 64) starts at offset off0 of page p0 and,
// when it runs past the page end T, continues at offset 0 of page p1.  T >= 64
// for frame pages, so a tile touches at most two pages.  Contiguous (text)
// keys behave as one unbounded page.
struct TileMap {
  const bf16_t* k0;   // key row of offset 0 in page p0 (this head)
  const bf16_t* k1;
  const bf16_t* v0;   // value column of offset 0 in page p0 (this head, dim 0)
  const bf16_t* v1;
  int off0;
  int T;
};

template <int HD, bool PAGED>
__device__ __forceinline__ TileMap map_tile(const AttnArgs& a, const AttnStream& S, int h, int j0) {
  TileMap m;
  if (PAGED) {
    const int32_t* pt = a.page_table + static_cast<size_t>(S.stream) * a.max_frames;
    const int fr = static_cast<int>(fdiv(static_cast<uint32_t>(j0), a.fT));
    m.off0 = j0 - fr * a.T;
    m.T = a.T;
    int p0 = pt[fr];
    p0 = p0 < 0 ? 0 : (p0 >= a.n_pages ? a.n_pages - 1 : p0);
    int p1 = p0;
    // the next page is read only when it holds keys of this stream
    if (m.off0 + BKV > a.T && (fr + 1) * a.T < S.kv_len) {
      p1 = pt[fr + 1];
      p1 = p1 < 0 ? 0 : (p1 >= a.n_pages ? a.n_pages - 1 : p1);
    }
    const size_t hs = static_cast<size_t>(a.T) * HD;
    m.k0 = a.k + (static_cast<size_t>(p0) * a.H + h) * hs;
    m.k1 = a.k + (static_cast<size_t>(p1) * a.H + h) * hs;
    m.v0 = a.v + (static_cast<size_t>(p0) * a.H + h) * hs;
    m.v1 = a.v + (static_cast<size_t>(p1) * a.H + h) * hs;
  } else {
    const size_t hs = static_cast<size_t>(S.T) * HD;
    m.k0 = m.k1 = a.k + static_cast<size_t>(S.base_off) + h * hs;
    m.v0 = m.v1 = a.v + static_cast<size_t>(S.base_off) + h * hs;
    m.off0 = j0;
    m.T = 0x7fffffff;   // never crossed
  }
  return m;
}

// Normalised bf16 output of one item.
template <int HD>
__device__ __forceinline__ void store_output(const AttnArgs& a, const AttnStream& S, int h, int qt,
                                             const f32x4 (&o)[2][HD / 16], const float (&l_run)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float l_tot = rows4_sum(l_run[qb]);
    const float inv = 1.0f / l_tot;
    const int ql = qt * BQ + wave * 32 + 16 * qb + l16;
    if (ql < S.q_len) {
      bf16_t* op = a.o + static_cast<size_t>(S.q_off + ql) * a.ldo + h * HD;
#pragma unroll
      for (int db = 0; db < HD / 16; ++db) {
        uint2 w;
        w.x = pack_bf16x2(o[qb][db][0] * inv, o[qb][db][1] * inv);
        w.y = pack_bf16x2(o[qb][db][2] * inv, o[qb][db][3] * inv);
        *reinterpret_cast<uint2*>(op + 16 * db + 4 * g) = w;
      }
    }
  }
}

// Partial results of a piece of a split item into slot `slot`: fp32 o, running
// max and denominator per query row of the item.
template <int HD>
__device__ __forceinline__ void store_partial(const AttnArgs& a, size_t slot,
                                              const f32x4 (&o)[2][HD / 16],
                                              const float (&m_run)[2], const float (&l_run)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float l_tot = rows4_sum(l_run[qb]);
    const int row = wave * 32 + 16 * qb + l16;
    float* po = a.part_o + (slot * BQ + row) * HD;
#pragma unroll
    for (int db = 0; db < HD / 16; ++db)
      *reinterpret_cast<float4*>(po + 16 * db + 4 * g) =
          make_float4(o[qb][db][0], o[qb][db][1], o[qb][db][2], o[qb][db][3]);
    if (g == 0) {
      a.part_ml[slot * 2 * BQ + row] = m_run[qb];
      a.part_ml[slot * 2 * BQ + BQ + row] = l_tot;
    }
  }
}

// Runs key tiles [tb, te) of item (S, head h, query tile qt) over the
// workgroup's 256 queries, then writes the normalised output (slot < 0) or
// the partial results into slot `slot`.  LIST: positions [tb, te) index the
// tile list tl (block-sparse attention) instead of being the tiles themselves.
//
// What bounds it: the matrix pipe (64 MFMAs of 16 clocks a wave and tile), the
// issue port that MFMAs (8 clocks each) and vector instructions (4; exponentials
// 8) share, at a clock that the card lowers under the load (2.15 GHz of 2.4 over
// 32760 keys of 12 heads, 1.95 over 37440 of 40, with the matrix cores busy 54 and
// 60% of it: a large product keeps them 91% busy at 1.72).  Two waves share a SIMD, w and
// w + 4.  When all eight met at a barrier every tile they ran in step: both in
// the products, then both in the softmax, about 4000 clocks a tile where the
// products take 2048.  So the two halves of the workgroup are a half tile
// apart.  A position's work is an MFMA phase (O += V P of the position before,
// then S = K Q: no softmax in between) and a VALU phase (its softmax, and the
// requests for tiles to come); each wave meets one barrier a position, group 0
// before its MFMA phase and group 1 before its VALU phase, so between two
// barriers one group runs MFMA then VALU and the other VALU then MFMA.
// s_setprio lets the MFMA phase issue first: its partner's vector instructions
// fit in the other half of the port.
// Tiles arrive by direct global -> LDS loads (no registers: with the staged
// tiles in them the loop spilled, and every reload waited for the tiles in
// flight) into four slots each, as pairs: pair u is the keys of position u and
// the values of u - 1.  Interval t (after barrier t) reads pair t and requests
// pair t + 3, whose slots were last read in interval t - 1; pair t + 1 is
// waited for before barrier t + 1.  Page ids and list entries of 64 frames or
// positions ride in one vector register, a lane each, so that the loop makes no
// scalar load: an LDS wait would have to cover it.
// Measured, in turn on one card: 4680 queries over 14040 keys, 12 heads, 386 ->
// 348 us; over 37440 keys, 20 heads, 2010 -> 1770; the 1.3B-class block step 1405
// -> 1290, the large one 6060 -> 5640; two barriers a tile (a strict exchange of
// phases) 352 / 1780 / 1295 / 5650; without s_setprio 1-2% slower.  Reading six
// or eight fragments ahead instead of four, or one branch for both query
// blocks' rescaling, changed nothing.
template <int HD, bool PAGED, bool VEC, bool LIST = false>
__device__ __forceinline__ void attn_range(const AttnArgs& a, const AttnStream& S, int h, int qt,
                                           int tb, int te, bf16_t (&sK)[NSLOT * BKV * HD],
                                           bf16_t (&sV)[NSLOT * HD * BKV], int64_t slot,
                                           const int32_t* tl = nullptr) {
  constexpr int KLD = HD;              // LDS row of the key tile
  constexpr int VLD = BKV;             // LDS row of the value tile
  constexpr int TILE = BKV * HD;       // elements of a key or value tile
  constexpr int NI = TILE * 2 / 1024 / 8;   // 1 KB loads per wave of a key or value tile
  constexpr int KS = HD / 32;          // 16x16x32 MFMA k-steps over d
  constexpr int DB = HD / 16;          // 16-wide output blocks over d
  static_assert(4 * KS >= LDS_AHEAD && 2 * DB >= LDS_AHEAD && NTHR == 512, "tile shape");
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int grp = wave >> 2;   // waves w and w + 4 share a SIMD: one of each group
  const int n = te - tb;

  // fragment read offsets: rows kb * 16 + l16 / db * 16 + l16 share the swizzle of l16
  int k_frag[KS], v_frag[2];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_frag[ks] = l16 * KLD + 8 * ((4 * ks + g) ^ swz<HD * 2>(l16));
#pragma unroll
  for (int ps = 0; ps < 2; ++ps) v_frag[ps] = l16 * VLD + 8 * ((4 * ps + g) ^ swz<BKV * 2>(l16));
  const float c = a.scale_log2;

  // ---- Q fragments (B operand of S^T = K Q^T): the wave's 32 rows are two
  // 16-row blocks; lane holds row l16 of block qb, dims 32 ks + 8 g ..
  bf16x8 qf[2][KS];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int q_row = min(qt * BQ + wave * 32 + 16 * qb + l16, S.q_len - 1);
    const bf16_t* qp = a.q + static_cast<size_t>(S.q_off + q_row) * a.ldq + h * HD;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[qb][ks] = *reinterpret_cast<const bf16x8*>(qp + 32 * ks + 8 * g);
  }

  const int kv_len = S.kv_len;
  const int vstride = PAGED ? a.T : S.T;   // distance between value dims
  const int nfull = kv_len / BKV;          // tiles whose 64 keys are all valid

  f32x4 o[2][DB];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[qb][db][v] = 0.f;
  // running max (scaled, log2) of the lane's rows; it starts finite, so that a piece
  // whose scores all overflow to -inf weighs nothing in the merge (-inf - -inf is NaN)
  float m_run[2] = {kNoMax, kNoMax};
  float l_run[2] = {0.f, 0.f};               // this lane's quarter of each running denominator
  f32x4 s[4][2];
  bf16x8 pf[2][2];

  // ---- staging.  Load j of this wave fills LDS rows of 1 KB: of a key tile the
  // rows R0 .. R0 + 1024 / (2 HD), R0 = (wave NI + j) 1024 / (2 HD), lane i the
  // 16-byte slot i % CPR of its row, which holds chunk (i % CPR) ^ swz(row) of
  // key kappa(row); of a value tile dims 8 (wave + 8 j) .. + 8, lane i slot
  // i % 8 of dim i / 8, chunk (i % 8) ^ swz(dim) (the same for every j).
  constexpr int CPR = HD / 8;
  constexpr int KROWS = 64 / CPR;
  uint32_t k_off[NI];       // byte offset from the tile's first key
  int k_key[NI];            // first key of the load's rows (d = 128: 4 aligned keys, one page)
  int k_lane_key[NI];       // this lane's key (d = 64: the rows may lie in two pages)
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int R = (wave * NI + j) * KROWS + lane / CPR;
    const int key = kappa16(R >> 4, R & 15);
    k_lane_key[j] = key;
    k_key[j] = kappa16((wave * NI + j) * KROWS >> 4, (wave * NI + j) * KROWS & 15);
    k_off[j] = static_cast<uint32_t>(key * HD * 2 + ((lane % CPR) ^ swz<HD * 2>(R & 15)) * 16);
  }
  const int v_dim = 8 * wave + (lane >> 3);
  const int v_key = 8 * ((lane & 7) ^ swz<BKV * 2>(v_dim));   // first key of this lane's chunk
  const uint32_t v_off = static_cast<uint32_t>((v_dim * vstride + v_key) * 2);
  const uint32_t lds_k = lds_address(sK) + wave * NI * 1024u, lds_v = lds_address(sV) + wave * 1024u;

  const int last_frame = PAGED ? min(static_cast<int>(fdiv(static_cast<uint32_t>(kv_len - 1), a.fT)),
                                     a.max_frames - 1) : 0;
  const int32_t* pt = PAGED ? a.page_table + static_cast<size_t>(S.stream) * a.max_frames : nullptr;
  // lane i: page of frame f0 + i, clamped into the pool
  auto page_window = [&](int f0) __attribute__((always_inline)) {
    const int p = pt[min(f0 + lane, last_frame)];
    return p < 0 ? 0 : (p >= a.n_pages ? a.n_pages - 1 : p);
  };
  // lane i: list entry b0 + i; entries are clamped into the stream's tiles, so a
  // corrupt list cannot send the loads outside the pages
  auto list_window = [&](int b0) __attribute__((always_inline)) {
    return min(max(tl[tb + min(b0 + lane, n - 1)], 0), S.n_tiles - 1);
  };
  const size_t hs = static_cast<size_t>(PAGED ? a.T : S.T) * HD;
  int lw0 = 0, lw = 0;
  if (LIST) lw = list_window(0);
  const size_t page_bytes = 2 * hs * a.H;   // of keys, and of values
  const char* k_head = reinterpret_cast<const char*>(a.k + h * hs);
  const char* v_head = reinterpret_cast<const char*>(a.v + h * hs);
  int fr = -2, pw0 = 0, pw = 0;   // (-2: no frame, nor the one before frame 0)
  const char *kp0 = nullptr, *kp1 = nullptr, *vp0 = nullptr, *vp1 = nullptr;
  if (PAGED) {
    // (a stream of up to 64 frames needs one window, which does not wait for the list)
    if (last_frame >= 64) {
      const int first = LIST ? __builtin_amdgcn_readlane(lw, 0) : tb;
      pw0 = static_cast<int>(fdiv(static_cast<uint32_t>(first * BKV), a.fT));
    }
    pw = page_window(pw0);
  } else {
    kp0 = kp1 = reinterpret_cast<const char*>(a.k + static_cast<size_t>(S.base_off) + h * hs);
    vp0 = vp1 = reinterpret_cast<const char*>(a.v + static_cast<size_t>(S.base_off) + h * hs);
  }
  const char* v_prev = nullptr;   // this lane's value address of the position moved to last
  int off0 = 0;
  // tile of the position moved to last: a list's entry read again for the values of the
  // first and last pairs was a trip to memory each (14040 keys of 12 heads 347.5 ->
  // 344.5 us, 52 kept tiles of 512 with their selection 138.7 -> 137.5)
  int id = tb;
  // moves to position u < n: tile, page bases, off0
  auto move_to = [&](int u) __attribute__((always_inline)) {
    id = tb + u;
    if (LIST) {
      if (u - lw0 >= 64) {
        lw0 = u;
        lw = list_window(u);
        asm volatile("" : "+v"(lw));   // waited for here, so no later wait has to
      }
      id = __builtin_amdgcn_readlane(lw, u - lw0);
    }
    const int j0 = id * BKV;
    off0 = j0;
    if (PAGED) {
      const int f = static_cast<int>(fdiv(static_cast<uint32_t>(j0), a.fT));
      off0 = j0 - f * a.T;
      if (f != fr) {   // bases of frame f and the next, less the next's offset
        if (f + 1 - pw0 >= 64) {
          pw0 = f;
          pw = page_window(f);
          asm volatile("" : "+v"(pw));
        }
        // One product a page, and over consecutive frames one page a frame: where a
        // frame is a tile or two long this runs every tile, and with the eight 64-bit
        // scalar products of both pages' keys and values 2500 queries over 14596 keys,
        // 20 heads of 64, frames of 64, took 320 us for 311.
        if (!LIST && f == fr + 1) {
          kp0 = kp1 + 2 * hs;
          vp0 = vp1 + 2 * a.T;
        } else {
          const size_t p0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(pw, f - pw0)) * page_bytes;
          kp0 = k_head + p0;
          vp0 = v_head + p0;
        }
        const size_t p1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(pw, f + 1 - pw0)) * page_bytes;
        kp1 = k_head + p1 - 2 * hs;
        vp1 = v_head + p1 - 2 * a.T;
        fr = f;
      }
    }
  };
  // direct loads of the keys of the current position into slot u % NSLOT, and of
  // the values of the position before into slot (u - 1) % NSLOT
  auto dma_keys = [&](int u) __attribute__((always_inline)) {
    const uint32_t dst = lds_k + static_cast<uint32_t>(u % NSLOT) * (TILE * 2);
    const ptrdiff_t ko = static_cast<ptrdiff_t>(off0) * (2 * HD);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      if constexpr (HD == 128) {
        const char* b = (PAGED && off0 + k_key[j] >= a.T ? kp1 : kp0) + ko;
        lds_dma16(b, k_off[j], dst + 1024u * j);
      } else {
        const char* b = (PAGED && off0 + k_lane_key[j] >= a.T ? kp1 : kp0) + ko;
        lds_dma16(b + k_off[j], dst + 1024u * j);
      }
    }
    const char* vb = (PAGED && off0 + v_key >= a.T ? vp1 : vp0) + 2 * static_cast<ptrdiff_t>(off0);
    v_prev = vb + v_off;
  };
  auto dma_values = [&](int u) __attribute__((always_inline)) {   // of position u
    const uint32_t dst = lds_v + static_cast<uint32_t>(u % NSLOT) * (TILE * 2);
#pragma unroll
    for (int j = 0; j < NI; ++j)
      lds_dma16(v_prev + static_cast<size_t>(j) * 128 * vstride, dst + 8192u * j);
  };
  // Base (text: p) that offset o_ of the current tile counts from, taken anew from
  // the page window; `over` bytes are one page's offsets.  (With kp0 .. vp1 used here
  // too, the d = 64 loop kept them in vector registers, 148 for 128 a lane: below.)
  auto tile_base = [&](const char* p, const char* head, int o_, size_t over) __attribute__((always_inline)) {
    if constexpr (!PAGED) return p;
    const size_t p0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(pw, fr - pw0)) * page_bytes;
    const size_t p1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(pw, fr + 1 - pw0)) * page_bytes;
    return head + (o_ >= a.T ? p1 - over : p0);
  };
  // Pair u: the keys of position u and the values of position u - 1.  At the
  // range's ends the last tile, when keys run out inside it, and text of odd
  // length go through registers, zeroed past the end.  (Lane indices are taken
  // anew there: shared with the main loop they would stay in registers across it.)
  // The partial tile comes in 16-byte pieces, NI trips to memory for its keys and
  // NI for its values.  Element by element, with the page
  // looked up again, its values took eight times as many, which only a long item
  // hides: on a split schedule, whose ranges are short, 480 queries over 5984 keys,
  // 12 heads, took 47.0 us for 44.9, and five streams of 720 over up to 5760, 9
  // heads, 147 for 132.  (With the two trips of d = 128 issued together the long
  // items' loop is up to 1% slower: other registers.)
  auto fetch = [&](int u) __attribute__((always_inline)) {
    if (u > 0 && u <= n) {
      // pairs are fetched in order: id, off0 and fr are those of the keys before
      // (move_to(u) comes after)
      if (VEC && id < nfull) {
        dma_values(u - 1);
      } else {
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));
        const int dim = 8 * wave + (ln >> 3), key = 8 * ((ln & 7) ^ swz<BKV * 2>(dim));
        const int left = kv_len - id * BKV - key, o_ = off0 + key;
        const bf16_t* vb = reinterpret_cast<const bf16_t*>(tile_base(vp0, v_head, o_, 2 * a.T)) + o_ +
                           static_cast<size_t>(dim) * vstride;
        bf16_t* dst = &sV[((u - 1) % NSLOT) * TILE + wave * 512 + ln * 8];
        if constexpr (VEC) {
          // pieces of 8 keys are 16-byte aligned, and one that holds a key lies whole in
          // its row of the page (or of the text): rows are multiples of 8 keys long
#pragma unroll 1
          for (int j = 0; j < NI; ++j) {
            u32x4 x = {0u, 0u, 0u, 0u};
            if (left > 0) x = *reinterpret_cast<const u32x4*>(vb + static_cast<size_t>(64 * j) * vstride);
#pragma unroll
            for (int i = 0; i < 4; ++i)   // (past the end the page may hold anything)
              x[i] = 2 * i + 1 < left ? x[i] : (2 * i < left ? x[i] & 0xffffu : 0u);
            *reinterpret_cast<u32x4*>(dst + j * 4096) = x;
          }
        } else {
          // Every tile comes this way when a text's length is no multiple of 8: all
          // its loads together (one after the other, a block step over 511 text
          // tokens took 669 us for 637, five streams of which two are odd 428 for 407).
          bf16_t x[NI][8];
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              x[j][e] = e < left ? vb[static_cast<size_t>(64 * j) * vstride + e] : bf16_t(0);
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[j * 4096 + e] = x[j][e];
        }
      }
    }
    if (u < n) {
      move_to(u);
      if (id < nfull) {
        dma_keys(u);
      } else {   // (a partial tile's values come with the next pair, through registers)
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));
#pragma unroll 1
        for (int j = 0; j < NI; ++j) {
          const int R = (wave * NI + j) * KROWS + ln / CPR;
          const int key = kappa16(R >> 4, R & 15), o_ = off0 + key;
          const bf16_t* b = reinterpret_cast<const bf16_t*>(tile_base(kp0, k_head, o_, 2 * hs)) +
                            static_cast<ptrdiff_t>(o_) * HD + 8 * ((ln % CPR) ^ swz<HD * 2>(R & 15));
          u32x4 x = {0u, 0u, 0u, 0u};
          if (id * BKV + key < kv_len) x = *reinterpret_cast<const u32x4*>(b);
          *reinterpret_cast<u32x4*>(&sK[(u % NSLOT) * TILE + (wave * NI + j) * 512 + ln * 8]) = x;
        }
      }
    }
  };

  // MFMA phase of position t: O^T += V^T P^T of position t - 1 (pv), then
  // S^T = K Q^T of position t (qk)
  auto mfma_phase = [&](int t, auto pv_c, auto qk_c) __attribute__((always_inline)) {
    constexpr bool PV = decltype(pv_c)::value, QK = decltype(qk_c)::value;
    bf16x8 vf[2][DB], kf[KS][4];
    __builtin_amdgcn_s_setprio(1);
    if constexpr (PV) {
      const bf16_t* tv = &sV[((t - 1) % NSLOT) * TILE];
#pragma unroll
      for (int ps = 0; ps < 2; ++ps)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          vf[ps][db] = *reinterpret_cast<const bf16x8*>(&tv[db * 16 * VLD + v_frag[ps]]);
#pragma unroll
      for (int ps = 0; ps < 2; ++ps)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
            o[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[ps][db], pf[qb][ps], o[qb][db], 0, 0, 0);
    }
    if constexpr (QK) {
      const bf16_t* tk = &sK[(t % NSLOT) * TILE];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int v = 0; v < 4; ++v) s[kb][qb][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
          kf[ks][kb] = *reinterpret_cast<const bf16x8*>(&tk[kb * 16 * KLD + k_frag[ks]]);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
            s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks][kb], qf[qb][ks], s[kb][qb], 0, 0, 0);
    }
    // schedule: LDS_AHEAD reads, then one read per pair of MFMAs
    constexpr int NR = (PV ? 2 * DB : 0) + (QK ? 4 * KS : 0);
    __builtin_amdgcn_sched_group_barrier(0x100, LDS_AHEAD, 0);
#pragma unroll
    for (int i = 0; i < NR - LDS_AHEAD; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * LDS_AHEAD, 0);
    __builtin_amdgcn_s_setprio(0);
    if constexpr (HD == 128) __builtin_amdgcn_sched_barrier(0);
  };

  // softmax of the scores of the current position into pf (ends: the position's
  // tile may hold keys past the end)
  auto softmax = [&](const bool ends, const int tile) __attribute__((always_inline)) {
    if (ends && tile >= nfull) {   // keys past the end (the last position only)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int key = tile * BKV + kappa16(kb, 4 * g + v);
          if (key >= kv_len) {
            s[kb][0][v] = -INFINITY;
            s[kb][1][v] = -INFINITY;
          }
        }
    }
    // online softmax in scaled log2 units; the running max is raised only when
    // a row's tile max exceeds it by more than 8 (p <= 2^8 otherwise), so the
    // O / l rescale is skipped on almost every tile
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v) mx = fmaxf(mx, s[kb][qb][v]);
      mx = rows4_max(mx) * c;
      if (__any(mx > m_run[qb] + 8.0f)) {
        const float m_new = fmaxf(m_run[qb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        m_run[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int v = 0; v < 4; ++v) o[qb][db][v] *= alpha;
      }
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const float mr = m_run[qb];
#pragma unroll
      for (int ps = 0; ps < 2; ++ps) {
        // keys 2 e2, 2 e2 + 1 of the step packed into one register, which both
        // feeds the P operand and is summed into the denominator (a plain
        // array: filling a 4-word vector element by element here compiled to
        // dot products that all read its first word)
        uint32_t pw[4];
        const bf16x2 one2 = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const int e = 2 * e2;
          const float p0 =
              __builtin_amdgcn_exp2f(fmaf(s[2 * ps + (e >> 2)][qb][e & 3], c, -mr));
          const float p1 = __builtin_amdgcn_exp2f(
              fmaf(s[2 * ps + ((e + 1) >> 2)][qb][(e + 1) & 3], c, -mr));
          pw[e2] = pack_bf16x2(p0, p1);
          l_run[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[e2]),
                                                      one2, l_run[qb], false);
        }
        pf[qb][ps] = __builtin_bit_cast(bf16x8, u32x4{pw[0], pw[1], pw[2], pw[3]});
      }
    }
    // The weights and sums are formed here, in this phase.  At d = 64 the MFMA phase
    // is half as long and cannot hide the whole softmax of the other group: there the
    // compiler may carry a part of it into the products that follow.
    if constexpr (HD == 128)
      asm volatile("" : "+v"(pf[0][0]), "+v"(pf[0][1]), "+v"(pf[1][0]), "+v"(pf[1][1]), "+v"(l_run[0]), "+v"(l_run[1]));
  };
  const std::true_type yes;
  const std::false_type no;

  // ---- prologue: the pairs ahead of the group's first VALU phase
#pragma unroll 1
  for (int u = 0; u < 3 + grp; ++u) fetch(u);
  if (!VEC || 2 + grp > n - 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else if (grp == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NI) : "memory");   // pair 0 has landed
  else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(6 * NI) : "memory");
  __syncthreads();
  const int last_tile = LIST ? min(max(tl[te - 1], 0), S.n_tiles - 1) : te - 1;
  // requests pair u
  auto stage = [&](int u) __attribute__((always_inline)) {
    if (VEC && u <= n - 2) {   // whole, and so are all before it
      dma_values(u - 1);
      move_to(u);
      dma_keys(u);
    } else {
      fetch(u);
    }
  };
  // the pair read after the next barrier has landed; u: the last pair requested
  auto wait_next = [&](int u) __attribute__((always_inline)) {
    if (VEC && u <= n - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NI) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  if (qt * BQ + wave * 32 < S.q_len) {
    mfma_phase(0, no, yes);
#pragma unroll 1
    for (int t = 0; t + 1 < n; ++t) {
      if (grp == 1) {
        wait_next(t + 3);
        __syncthreads();
      }
      stage(t + 3 + grp);
      softmax(false, 0);
      if (grp == 0) {
        wait_next(t + 3);
        __syncthreads();
      }
      mfma_phase(t + 1, yes, yes);
    }
    // The last position: nothing is left to request, and no scores follow (formed
    // over whatever the next slot held, they cost every range 0.4 us and more: 480
    // queries over 544 keys, 40 heads of 128, 25.6 us for 24.9; 2500 over 14596, 20
    // heads of 64, 327 for 320).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (grp == 1) __syncthreads();
    softmax(true, last_tile);
    if (grp == 0) __syncthreads();
    mfma_phase(n, yes, no);
  } else {   // no query of this wave exists: it only stages
#pragma unroll 1
    for (int t = 0; t < n; ++t) {
      if (grp == 0) stage(t + 3);
      wait_next(t + 3);
      __syncthreads();
      if (grp == 1) stage(t + 4);
    }
  }
  if (slot < 0)
    store_output<HD>(a, S, h, qt, o, l_run);
  else
    store_partial<HD>(a, static_cast<size_t>(slot), o, m_run, l_run);
  if (slot >= 0) __syncthreads();   // a following range reuses the tiles
}

// One workgroup per item.  At d = 64 past one round two workgroups share a CU (64 KB
// of LDS each), if a lane takes at most 128 registers: five streams of 3328 queries
// over 17728 keys, 20 heads, 2190 us with 148, 1760 so.  AttnArgs::alone keeps them
// apart (launch_attn_t).
template <int HD, bool PAGED, bool VEC>
__global__ __launch_bounds__(NTHR, HD == 64 ? 4 : 1) void attn_kernel(const AttnArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t sK[NSLOT * BKV * HD];
  __shared__ __attribute__((aligned(16))) bf16_t sV[NSLOT * HD * BKV];

  // ---- work item (XCD-aware: each XCD runs a contiguous range of items, so
  // the items of one head share its L2, the ranges balanced by tile count)
  const int pid = blockIdx.x;
  const int xcd = pid % kNumXcd;
  const int L = a.xcd_begin[xcd] + pid / kNumXcd;
  if (L >= a.xcd_begin[xcd + 1]) return;
  int si = 0;
  for (int i = 1; i < a.n_streams; ++i)
    if (L >= a.s[i].item_begin) si = i;
  const AttnStream S = a.s[si];
  const int it = L - S.item_begin;
  const int h = it / S.n_qtiles;
  const int qt = it - h * S.n_qtiles;
  attn_range<HD, PAGED, VEC>(a, S, h, qt, 0, S.n_tiles, sK, sV, -1);
}

// Split schedule: each item runs its first main_tiles tiles in its own
// workgroup; the remaining workgroups take equal ranges of the concatenated tails.
template <int HD, bool PAGED, bool VEC>
__global__ __launch_bounds__(NTHR, 1) void attn_split_kernel(const AttnArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t sK[NSLOT * BKV * HD];
  __shared__ __attribute__((aligned(16))) bf16_t sV[NSLOT * HD * BKV];

  const int pid = blockIdx.x;
  const int xcd = pid % kNumXcd, j = pid / kNumXcd;

  // XCD x runs items item0 + [pre, pre + nx), then its share of the tail ranges
  const int items = a.total_items - a.item0;
  const int ipx = items / kNumXcd, irem = items % kNumXcd;
  const int nx = ipx + (xcd < irem ? 1 : 0);
  const int pre = xcd * ipx + min(xcd, irem);
  if (j < nx) {
    const int gi = a.item0 + pre + j;
    int si = 0;
    for (int i = 1; i < a.n_streams; ++i)
      if (gi >= a.s[i].item_begin) si = i;
    const AttnStream S = a.s[si];
    const int item = gi - S.item_begin;
    const int h = item / S.n_qtiles, qt = item - h * S.n_qtiles;
    attn_range<HD, PAGED, VEC>(a, S, h, qt, 0, S.main_tiles, sK, sV,
                               S.main_tiles == S.n_tiles ? -1 : gi - a.item0);
    return;
  }
  const int r = a.per_xcd * xcd + j - (pre + nx);   // tail range
  if (r >= a.split_blocks - items) return;
  int pos = r * a.split_tiles;
  const int end = min(pos + a.split_tiles, a.total_tiles);
  while (pos < end) {
    int si = 0;
    for (int i = 1; i < a.n_streams; ++i)
      if (pos >= a.s[i].tail_begin) si = i;
    const AttnStream S = a.s[si];
    const int tl = S.n_tiles - S.main_tiles;
    const int rel = pos - S.tail_begin;
    const int first = max(0, a.item0 - S.item_begin);   // the stream's first item of this schedule
    const int item = first + rel / tl;
    const int tb = S.main_tiles + rel % tl;
    const int te = min(S.n_tiles, tb + (end - pos));
    pos += te - tb;
    const int h = item / S.n_qtiles, qt = item - h * S.n_qtiles;
    // piece (range r, item i) -> slot items + i + r: items increase within a
    // range and the next range starts at the last one's last item, so slots differ
    attn_range<HD, PAGED, VEC>(a, S, h, qt, tb, te, sK, sV,
                               static_cast<int64_t>(items) + S.item_begin + item - a.item0 + r);
  }
}

// Combines the partial results of the items that a split schedule cut:
// o = sum_j 2^(m_j - M) O_j / sum_j 2^(m_j - M) l_j, M = max_j m_j, over the
// item's main part (slot = item) and the pieces of its tail [w0, w1) of the
// concatenated tails, held by ranges w0 / W .. (w1 - 1) / W (slot
// items + item + range, items counted from item0).
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(const AttnArgs a) {
  constexpr int TPR = HD / 4;          // threads per row, 4 dims each
  constexpr int RPB = 256 / TPR;       // rows per workgroup
  const int gi = a.item0 + blockIdx.x / (BQ / RPB);
  const int row = (blockIdx.x % (BQ / RPB)) * RPB + threadIdx.x / TPR;
  int si = 0;
  for (int i = 1; i < a.n_streams; ++i)
    if (gi >= a.s[i].item_begin) si = i;
  const AttnStream& S = a.s[si];
  const int item = gi - S.item_begin;
  const int tl = S.n_tiles - S.main_tiles;
  if (tl == 0) return;   // written whole by its main part
  const int w0 = S.tail_begin + (item - max(0, a.item0 - S.item_begin)) * tl, w1 = w0 + tl;
  const int li = gi - a.item0, items = a.total_items - a.item0;
  const int W = a.split_tiles;
  const int b_lo = w0 / W, b_hi = (w1 - 1) / W;
  const int h = item / S.n_qtiles;
  const int qt = item - h * S.n_qtiles;
  const int d4 = threadIdx.x % TPR;
  const int ql = qt * BQ + row;
  if (ql >= S.q_len) return;
  {
    float M = a.part_ml[static_cast<size_t>(li) * 2 * BQ + row];
    for (int b = b_lo; b <= b_hi; ++b) {
      const size_t slot = static_cast<size_t>(items) + li + b;
      M = fmaxf(M, a.part_ml[slot * 2 * BQ + row]);
    }
    float l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int b = b_lo - 1; b <= b_hi; ++b) {
      const size_t slot = b < b_lo ? static_cast<size_t>(li) : static_cast<size_t>(items) + li + b;
      const float wgt = __builtin_amdgcn_exp2f(a.part_ml[slot * 2 * BQ + row] - M);
      l += wgt * a.part_ml[slot * 2 * BQ + BQ + row];
      const float4 p = *reinterpret_cast<const float4*>(a.part_o + (slot * BQ + row) * HD + 4 * d4);
      acc.x += wgt * p.x;
      acc.y += wgt * p.y;
      acc.z += wgt * p.z;
      acc.w += wgt * p.w;
    }
    const float inv = 1.0f / l;
    uint2 w;
    w.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    w.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2*>(a.o + static_cast<size_t>(S.q_off + ql) * a.ldo + h * HD + 4 * d4) = w;
  }
}

// Attention over few keys for few queries.  An item of attn_kernel walks its
// tiles one after the other (about 1.7 us each) on one CU, and small calls have
// a handful of items.  Here a workgroup takes 32 queries of one (stream, head)
// and its eight waves take every eighth key tile, so a call of H heads and q
// queries spreads over H q / 32 CUs and each wave walks n_tiles / 8 tiles.  A
// wave reads its K and V fragments straight from memory (the tiles are not
// shared between waves, so LDS would add a trip and two barriers), in the
// layouts attn_kernel reads from LDS; the waves' partial results meet in LDS at
// the end.  192 queries over 576 keys, 4 heads of 64 (the tiny block): 15.7 us
// on one workgroup per item, 8.6 here; 480 over 1440, 12 heads of 128: 46.8, 28.1.
// What bounds it is the chain of a wave's tiles: the fragment loads of one (32 KB in
// 64-byte pieces at d = 128) are issued together, but with K, V, O and Q in 256
// registers there is no room to ask for the next tile's.
constexpr int SM_BQ = 32;      // queries per workgroup
constexpr int SM_WAVES = 8;
// most key tiles of a stream (plan_attention)
constexpr int small_tiles(int head_dim) { return head_dim == 128 ? 31 : 47; }

template <int HD, bool PAGED, bool VEC>
__global__ __launch_bounds__(64 * SM_WAVES, 1) void attn_small_kernel(const AttnArgs a) {
  constexpr int KS = HD / 32, DB = HD / 16;
  __shared__ __attribute__((aligned(16))) float part[SM_WAVES][SM_BQ][HD];
  __shared__ float part_m[SM_WAVES][SM_BQ], part_l[SM_WAVES][SM_BQ];
  const int pid = blockIdx.x;
  const int L = (pid % kNumXcd) * a.per_xcd + pid / kNumXcd;
  if (L >= a.total_items) return;
  int si = 0;
  for (int i = 1; i < a.n_streams; ++i)
    if (L >= a.s[i].item_begin) si = i;
  const AttnStream S = a.s[si];
  const int it = L - S.item_begin;
  const int h = it / S.n_qtiles, qt = it - h * S.n_qtiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int kv_len = S.kv_len, vstride = PAGED ? a.T : S.T;
  const float c = a.scale_log2;

  bf16x8 qf[2][KS];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int q_row = min(qt * SM_BQ + 16 * qb + l16, S.q_len - 1);
    const bf16_t* qp = a.q + static_cast<size_t>(S.q_off + q_row) * a.ldq + h * HD;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *reinterpret_cast<const bf16x8*>(qp + 32 * ks + 8 * g);
  }
  f32x4 o[2][DB];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[qb][db][v] = 0.f;
  float m_run[2] = {kNoMax, kNoMax}, l_run[2] = {0.f, 0.f};

  for (int t = wave; t < S.n_tiles; t += SM_WAVES) {
    const int j0 = t * BKV;
    const TileMap tm = map_tile<HD, PAGED>(a, S, h, j0);
    bf16x8 kf[4][KS], vf[2][DB];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      // keys past the end read the stream's last key and are masked below
      const int o_ = min(tm.off0 + kappa16(kb, l16), tm.off0 + kv_len - 1 - j0);
      const bf16_t* p = o_ < tm.T ? tm.k0 + static_cast<size_t>(o_) * HD
                                  : tm.k1 + static_cast<size_t>(o_ - tm.T) * HD;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kb][ks] = *reinterpret_cast<const bf16x8*>(p + 32 * ks + 8 * g);
    }
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) {
      const int o_ = tm.off0 + 32 * ps + 8 * g, jv = j0 + 32 * ps + 8 * g;
      const bf16_t* vb = (o_ < tm.T ? tm.v0 + o_ : tm.v1 + (o_ - tm.T)) + static_cast<size_t>(l16) * vstride;
      const int left = kv_len - jv;
      if (VEC) {
        // A piece that holds a key lies whole in its row; past the end it may hold
        // anything.  (By element, one key took 7.1 us at d = 128, 5.2 this way.)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          u32x4 x = {0u, 0u, 0u, 0u};
          if (left > 0) x = *reinterpret_cast<const u32x4*>(vb + static_cast<size_t>(16 * db) * vstride);
          vf[ps][db] = __builtin_bit_cast(bf16x8, x);
        }
        if (j0 + BKV > kv_len) {
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            u32x4 x = __builtin_bit_cast(u32x4, vf[ps][db]);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = 2 * i + 1 < left ? x[i] : (2 * i < left ? x[i] & 0xffffu : 0u);
            vf[ps][db] = __builtin_bit_cast(bf16x8, x);
          }
        }
      } else {   // values past the end are zero
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (e < left)
              w[e >> 1] |= static_cast<uint32_t>(vb[static_cast<size_t>(16 * db) * vstride + e]) << (16 * (e & 1));
          vf[ps][db] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
        }
      }
    }
    f32x4 s[4][2];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) s[kb][qb][v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][ks], qf[qb][ks], s[kb][qb], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j0 + kappa16(kb, 4 * g + v) >= kv_len) s[kb][qb][v] = -INFINITY;
      }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int v = 0; v < 4; ++v) mx = fmaxf(mx, s[kb][qb][v]);
      const float m_new = fmaxf(m_run[qb], rows4_max(mx) * c);
      const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
      m_run[qb] = m_new;
      l_run[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[qb][db][v] *= alpha;
      bf16x8 pf[2];
#pragma unroll
      for (int ps = 0; ps < 2; ++ps) {
        uint32_t pw[4];
        const bf16x2 one2 = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const int e = 2 * e2;
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[2 * ps + (e >> 2)][qb][e & 3], c, -m_new));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[2 * ps + ((e + 1) >> 2)][qb][(e + 1) & 3], c, -m_new));
          pw[e2] = pack_bf16x2(p0, p1);
          l_run[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[e2]), one2, l_run[qb], false);
        }
        pf[ps] = __builtin_bit_cast(bf16x8, u32x4{pw[0], pw[1], pw[2], pw[3]});
      }
#pragma unroll
      for (int ps = 0; ps < 2; ++ps)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          o[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[ps][db], pf[ps], o[qb][db], 0, 0, 0);
    }
  }

  // merge: o = sum_w 2^(m_w - M) o_w / sum_w 2^(m_w - M) l_w (a wave without
  // tiles adds nothing)
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float l_tot = rows4_sum(l_run[qb]);
    const int row = 16 * qb + l16;
#pragma unroll
    for (int db = 0; db < DB; ++db)   // 16-byte chunks XOR-swizzled by row over the banks
      *reinterpret_cast<float4*>(&part[wave][row][4 * ((4 * db + g) ^ (l16 & 15))]) =
          make_float4(o[qb][db][0], o[qb][db][1], o[qb][db][2], o[qb][db][3]);
    if (g == 0) {
      part_m[wave][row] = m_run[qb];
      part_l[wave][row] = l_tot;
    }
  }
  __syncthreads();
  for (int i = tid; i < SM_BQ * HD / 4; i += 64 * SM_WAVES) {
    const int row = i / (HD / 4), c4 = i % (HD / 4);
    const int ql = qt * SM_BQ + row;
    if (ql >= S.q_len) continue;
    float M = part_m[0][row];
#pragma unroll
    for (int w = 1; w < SM_WAVES; ++w) M = fmaxf(M, part_m[w][row]);
    float l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < SM_WAVES; ++w) {
      if (w >= S.n_tiles) break;   // (that wave had no tile)
      const float wgt = __builtin_amdgcn_exp2f(part_m[w][row] - M);
      const float4 p = *reinterpret_cast<const float4*>(&part[w][row][4 * (c4 ^ (row & 15))]);
      l += wgt * part_l[w][row];
      acc.x += wgt * p.x;
      acc.y += wgt * p.y;
      acc.z += wgt * p.z;
      acc.w += wgt * p.w;
    }
    const float inv = 1.0f / l;
    uint2 w;
    w.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    w.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2*>(a.o + static_cast<size_t>(S.q_off + ql) * a.ldo + h * HD + 4 * c4) = w;
  }
}

// Block-sparse attention: one workgroup per item over the item's kept tiles,
// read from its list (written by the block selection).
template <int HD>
__global__ __launch_bounds__(NTHR, 1) void attn_sparse_kernel(const AttnArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t sK[NSLOT * BKV * HD];
  __shared__ __attribute__((aligned(16))) bf16_t sV[NSLOT * HD * BKV];
  const int pid = blockIdx.x;
  const int xcd = pid % kNumXcd;
  const int L = a.xcd_begin[xcd] + pid / kNumXcd;
  if (L >= a.xcd_begin[xcd + 1]) return;
  int si = 0;
  for (int i = 1; i < a.n_streams; ++i)
    if (L >= a.s[i].item_begin) si = i;
  const AttnStream S = a.s[si];
  const int it = L - S.item_begin;
  const int h = it / S.n_qtiles;
  const int qt = it - h * S.n_qtiles;
  const int ld = a.blk_ld ? a.blk_ld : S.n_keep;
  const int32_t* tl = a.blocks + S.blk_off + static_cast<int64_t>(it) * ld;
  attn_range<HD, true, true, true>(a, S, h, qt, 0, S.n_keep, sK, sV, -1, tl);
}

}  // namespace

hipError_t launch_sparse_attention(hipStream_t st, const AttnArgs& a, int head_dim) {
  if (a.total_items == 0) return hipSuccess;
  const dim3 grid(a.per_xcd * kNumXcd);
  if (head_dim == 128)
    hipLaunchKernelGGL((attn_sparse_kernel<128>), grid, dim3(NTHR), 0, st, a);
  else if (head_dim == 64)
    hipLaunchKernelGGL((attn_sparse_kernel<64>), grid, dim3(NTHR), 0, st, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {

constexpr int kCusPerXcd = 32;   // MI355X: 8 XCDs of 32 CUs

// Item costs in plan order as runs: the items of one stream are contiguous
// and cost the same (its key tiles, or its kept tiles when sparse), so run r
// covers items [begin[r], begin[r + 1]) at cost[r].
struct CostRuns {
  int n;
  int32_t begin[kMaxStreams + 1];
  int32_t cost[kMaxStreams];
};

// List schedule of items [i, n) (plan order) onto one XCD's CUs, each CU
// taking the next item when it frees (how the dispatcher hands out an XCD's
// workgroups in order, one 512-thread workgroup per CU).  Returns the first
// item past those that finish by makespan M; with share > 0 it also stops once
// the XCD's cost reaches share.
int fill_xcd(const CostRuns& c, int i, int n, int64_t M, int64_t share) {
  int64_t fin[kCusPerXcd] = {};
  int64_t taken = 0;
  int r = 0;
  while (r + 1 < c.n && i >= c.begin[r + 1]) ++r;
  for (; i < n; ++i) {
    while (i >= c.begin[r + 1]) ++r;
    const int64_t cost = c.cost[r];
    if (share > 0 && taken >= share) break;
    int k = 0;
    for (int u = 1; u < kCusPerXcd; ++u) k = fin[u] < fin[k] ? u : k;
    if (fin[k] + cost > M) break;
    fin[k] += cost;
    taken += cost;
  }
  return i;
}

int64_t runs_cost(const CostRuns& c, int i0, int i1) {
  int64_t t = 0;
  for (int r = 0; r < c.n; ++r) {
    const int lo = c.begin[r] > i0 ? c.begin[r] : i0;
    const int hi = c.begin[r + 1] < i1 ? c.begin[r + 1] : i1;
    if (hi > lo) t += static_cast<int64_t>(hi - lo) * c.cost[r];
  }
  return t;
}

// Contiguous split of the items over the XCDs that minimises the makespan of
// the slowest XCD under list scheduling (binary search on the makespan), with
// the items spread evenly by cost where that makespan allows.  Returns the makespan.
int64_t split_by_makespan(const CostRuns& c, int n, int64_t total, int32_t* begin) {
  int64_t lo = 0, hi = total;
  for (int r = 0; r < c.n; ++r)
    if (c.begin[r + 1] > c.begin[r]) lo = c.cost[r] > lo ? c.cost[r] : lo;
  auto feasible = [&](int64_t M) {
    int i = 0;
    for (int x = 0; x < kNumXcd && i < n; ++x) i = fill_xcd(c, i, n, M, 0);
    return i == n;
  };
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (feasible(mid)) hi = mid;
    else lo = mid + 1;
  }
  // even spread first, bounded by the makespan; the greedy fill if that fails
  for (int pass = 0; pass < 2; ++pass) {
    int i = 0;
    int64_t done = 0;
    begin[0] = 0;
    for (int x = 0; x < kNumXcd; ++x) {
      int64_t share = 0;
      if (pass == 0 && x < kNumXcd - 1) {
        share = (total - done) / (kNumXcd - x);
        share = share > 0 ? share : 1;
      }
      const int e = fill_xcd(c, i, n, lo, share);
      done += runs_cost(c, i, e);
      i = e;
      begin[x + 1] = i;
    }
    if (i == n) return lo;
  }
  return lo;
}

// The last plans' XCD splits, reused while the item costs repeat (every layer
// and denoising step of a chunk has the same geometry).  A block plans two
// attentions, self and text, and a chunk's passes shrink as streams finish:
// with one entry the two replaced each other and every block call searched both
// again, 440 us of host time at the 1.3B-class shape (now 45).  Fixed-size and per
// thread, so planning makes no host allocation and takes no lock.
constexpr int kXcdSplitEntries = 8;
struct XcdSplitCache {
  struct Entry {
    int32_t key[2 * kMaxStreams + 1];
    int key_len = -1;
    int32_t begin[kNumXcd + 1];
    int32_t alone;
  } e[kXcdSplitEntries];
  int next = 0;   // the entry replaced next
};

}  // namespace

void balance_items_over_xcds(AttnArgs& a, bool sparse) {
  // per-stream item runs in plan order, also the cache key
  thread_local XcdSplitCache cache;
  int32_t key[2 * kMaxStreams + 1];
  int key_len = 0;
  key[key_len++] = a.H;
  CostRuns runs;
  runs.n = a.n_streams;
  int64_t total = 0;
  for (int i = 0; i < a.n_streams; ++i) {
    const int32_t c = sparse ? a.s[i].n_keep : a.s[i].n_tiles;
    key[key_len++] = a.s[i].n_qtiles;
    key[key_len++] = c;
    runs.begin[i] = a.s[i].item_begin;
    runs.cost[i] = c;
    total += static_cast<int64_t>(a.s[i].n_qtiles) * a.H * c;
  }
  const int n = a.total_items;
  runs.begin[a.n_streams] = n;
  int64_t longest = 0;
  for (int i = 0; i < a.n_streams; ++i) longest = runs.cost[i] > longest ? runs.cost[i] : longest;
  const XcdSplitCache::Entry* hit = nullptr;
  for (const XcdSplitCache::Entry& c : cache.e)
    if (c.key_len == key_len && memcmp(key, c.key, sizeof(int32_t) * static_cast<size_t>(key_len)) == 0) {
      hit = &c;
      break;
    }
  if (!hit) {
    XcdSplitCache::Entry& c = cache.e[cache.next];
    cache.next = (cache.next + 1) % kXcdSplitEntries;
    c.alone = 0;
    if (n <= 65536) {
      const int64_t end = split_by_makespan(runs, n, total, c.begin);
      // Two workgroups of a CU run at about 0.6 of the speed of one each.  That
      // delays the end where the longest items take the whole time by themselves, all
      // others fit beside them and little room is left.  us together and apart, d = 64,
      // 4672 queries, 8 heads: streams of 512 and 220 tiles 712 / 658; of 512 and 80
      // (a third of the room left) 660 / 657; of 512 and 440 (two rounds) 981 / 1129;
      // 10 heads, 192 and 73 265 / 346.
      c.alone = 32 * end <= 33 * longest && 10 * kNumXcd * kCusPerXcd * end <= 13 * total;
    } else {   // very large batches: equal item counts
      for (int x = 0; x <= kNumXcd; ++x)
        c.begin[x] = static_cast<int32_t>(static_cast<int64_t>(n) * x / kNumXcd);
    }
    memcpy(c.key, key, sizeof(int32_t) * static_cast<size_t>(key_len));
    c.key_len = key_len;
    hit = &c;
  }
  int most = 0;
  a.alone = hit->alone;
  for (int x = 0; x <= kNumXcd; ++x) a.xcd_begin[x] = hit->begin[x];
  for (int x = 0; x < kNumXcd; ++x)
    most = a.xcd_begin[x + 1] - a.xcd_begin[x] > most ? a.xcd_begin[x + 1] - a.xcd_begin[x] : most;
  a.per_xcd = most;
}

size_t attention_split_bytes(int head_dim) {
  return static_cast<size_t>(2) * kAttnSplitBlocks * BQ * (head_dim + 2) * sizeof(float);
}

namespace {

// When a split schedule ends, in 128ths of a tile after the time of a whole item
// without its tiles.  A range's pieces after the first cost a start and a partial
// store each (5 tiles, about 7 us, at d = 128; 2.5, 3 us, at d = 64), every schedule the
// merge's launch, and every partial tile its trip to memory and back.  Fitted to 464
// calls of one round or less (8 to 200 items of 11 to 120 tiles), each timed whole and
// split; the rule takes the slower side by at most 5% in any of them.  Before it every
// round cut below 256 workgroups was split, and the short tails of items of 11 to 15
// tiles put two and three pieces into a range: us whole and split, d = 128: 36 items
// of 14 tiles 28.8 / 43.6, 176 of 11 27.9 / 49.5, streams of 4 to 31 tiles, 100
// items, 53.0 / 85.0; 36 items of 16, one piece a range, 31.5 / 29.1; of 18, two, 34.1 /
// 36.9; of 24, two, 42.4 / 37.9.
int64_t split_end(const AttnStream* s, int n, int split_tiles, int64_t tails, int head_dim) {
  const int64_t S = split_tiles;
  int32_t pieces[kAttnSplitBlocks] = {};   // of each tail range
  int64_t parts = 0;
  int longest = 0;
  for (int i = 0; i < n; ++i) {
    longest = max(longest, s[i].main_tiles);
    const int tl = s[i].n_tiles - s[i].main_tiles;
    const int64_t t0 = s[i].tail_begin, t1 = i + 1 < n ? s[i + 1].tail_begin : tails;
    if (t0 == t1) continue;
    parts += (t1 - t0) / tl;   // main parts
    for (int64_t r = t0 / S; r * S < t1; ++r) {
      const int64_t lo = max(r * S, t0) - t0, hi = min((r + 1) * S, t1) - t0;
      const int c = static_cast<int>((hi - 1) / tl - lo / tl + 1);
      pieces[r] += c;
      parts += c;
    }
  }
  int most = 0;
  for (int r = 0; r < kAttnSplitBlocks; ++r) most = max(most, pieces[r]);
  const bool wide = head_dim == 128;
  const int64_t last = 128 * S + (wide ? 640 : 320) * (most - 1);
  return max(static_cast<int64_t>(128) * longest, last) + (wide ? 640 + 2 * parts : 384 + 3 * parts);
}

}  // namespace

void plan_attention(AttnArgs& a, int head_dim, float* split_ws) {
  // order streams by decreasing key count so the longest items start first
  AttnStream tmp[kMaxStreams];
  int n = 0;
  for (int i = 0; i < a.n_streams; ++i)
    if (a.s[i].q_len > 0) tmp[n++] = a.s[i];
  for (int i = 1; i < n; ++i) {
    AttnStream x = tmp[i];
    int j = i - 1;
    while (j >= 0 && tmp[j].kv_len < x.kv_len) {
      tmp[j + 1] = tmp[j];
      --j;
    }
    tmp[j + 1] = x;
  }
  int items = 0;
  int64_t work = 0;
  for (int i = 0; i < n; ++i) {
    tmp[i].n_qtiles = (tmp[i].q_len + BQ - 1) / BQ;
    tmp[i].n_tiles = (tmp[i].kv_len + BKV - 1) / BKV;
    tmp[i].main_tiles = tmp[i].n_tiles;
    tmp[i].tail_begin = 0;
    tmp[i].item_begin = items;
    items += tmp[i].n_qtiles * a.H;
    work += static_cast<int64_t>(tmp[i].n_qtiles) * a.H * tmp[i].n_tiles;
  }
  a.n_streams = n;
  a.total_items = items;
  a.small = 0;
  a.alone = 0;
  a.item0 = 0;
  a.total_tiles = 0;
  a.split_blocks = 0;
  a.split_tiles = 0;
  a.part_o = nullptr;
  a.part_ml = nullptr;
  // Few queries over few keys: 32-query workgroups while they fit one round of
  // the CUs and the longest stream has so few tiles that a wave's share of them
  // takes no longer than the split schedule below, whose pieces have eight tiles
  // each and a merge behind them: up to 31 tiles at d = 128, 47 at d = 64.  us here
  // and split, d = 128: 192 queries, 12 heads, 16 tiles 21.4 / 24.4, 28 32.1 / 33.8,
  // 32 36.4 / 26.7, 64 66.2 / 30.8; 40 heads, 28 33.5 / 36.3, 32 37.2 / 29.1, 64
  // 66.6 / 44.3; 1024, 8 heads, 28 32.9 / 39.9, 32 36.9 / 33.2, 64 66.3 / 35.6.  d =
  // 64: 192, 20 heads, 40 22.9 / 28.1, 48 26.3 / 23.7, 64 33.3 / 26.4.  With items
  // that neither splits: 240 workgroups (40 heads, 192 queries) 9 tiles 16.5 for
  // 22.4.  Past one round it loses: 480 workgroups 52 us for 36 (60 tiles), 576: 84
  // for 49 (24).
  {
    int64_t wgs = 0;
    int most = 0;
    for (int i = 0; i < n; ++i) {
      wgs += static_cast<int64_t>((tmp[i].q_len + SM_BQ - 1) / SM_BQ) * a.H;
      most = tmp[i].n_tiles > most ? tmp[i].n_tiles : most;
    }
    if (items > 0 && wgs <= kAttnSplitBlocks && most <= small_tiles(head_dim)) {
      a.small = 1;
      a.total_items = static_cast<int32_t>(wgs);
      a.per_xcd = (a.total_items + kNumXcd - 1) / kNumXcd;
      int begin = 0;
      for (int i = 0; i < n; ++i) {
        tmp[i].n_qtiles = (tmp[i].q_len + SM_BQ - 1) / SM_BQ;
        tmp[i].item_begin = begin;
        begin += tmp[i].n_qtiles * a.H;
        a.s[i] = tmp[i];
      }
      return;
    }
  }
  // Split when the items fit one round of workgroups but leave more than a
  // quarter of them idle: every item keeps its first W tiles (W = the even
  // share of all tiles per workgroup) and the idle workgroups take equal ranges
  // of the remaining tails.  Items of one head still run their main parts in
  // step, sharing key tiles through L2.  The tail ranges cost more per tile (short
  // segments, partial writes, the merge) and end last, which outweighs the gain
  // while few workgroups are idle.  Whole and split, us at d = 128: 28 idle (228
  // items) 78 tiles 125 / 191, 220 330 / 396, 512 765 / 817; 56 idle 78 120 / 151,
  // 220 320 / 332, 313 455 / 450, 512 739 / 709; 64 idle 78 120 / 129, 128 188 /
  // 191, 220 316 / 304, 512 732 / 668.  (So from about a quarter idle on it depends
  // on the tiles too: split_end.)  The round is cut to as many workgroups as have
  // eight tiles each (a multiple of the XCDs; 1440 queries over 4320 keys, 4 heads
  // of 64, 1632 tiles on 24 items: 92 us unsplit, 34 on 200 workgroups).
  //
  // Items of equal cost that fill one to three rounds and leave more than a
  // quarter of the last one idle run their full rounds whole and split the rest
  // the same way in a second launch: 380 items of 585 tiles (4680 queries over
  // 37440 keys, 20 heads) 1520 us for 1770.  The launch and the merge take
  // about 20 us, so the idle share has to be worth 24 tiles of the round; with
  // more rounds, or with mixed costs (where shorter items fill the gaps), it is
  // not.
  const bool uniform = n > 0 && tmp[0].n_tiles == tmp[n - 1].n_tiles;   // (ordered by cost)
  int item0 = 0;
  if (items > kAttnSplitBlocks) {
    const int rem = items % kAttnSplitBlocks;
    const int idle = kAttnSplitBlocks - rem;
    if (!uniform || rem == 0 || items > 4 * kAttnSplitBlocks ||
        static_cast<int64_t>(idle) * tmp[0].n_tiles < 24 * kAttnSplitBlocks)
      item0 = items;
    else
      item0 = items - rem;
    work = item0 < items ? static_cast<int64_t>(rem) * tmp[0].n_tiles : 0;
  }
  const int left = items - item0;   // items to split
  const int blocks = static_cast<int>(min(static_cast<int64_t>(kAttnSplitBlocks), work / 8 / kNumXcd * kNumXcd));
  const int spare = blocks - left;
  if (split_ws && left > 0 && spare * 4 > blocks && work < (static_cast<int64_t>(1) << 30)) {
    const int W = static_cast<int>((work + blocks - 1) / blocks);
    int64_t tails = 0;
    for (int i = 0; i < n; ++i) {
      tmp[i].main_tiles = min(tmp[i].n_tiles, W);
      tmp[i].tail_begin = static_cast<int32_t>(tails);
      const int here = tmp[i].n_qtiles * a.H - min(tmp[i].n_qtiles * a.H, max(0, item0 - tmp[i].item_begin));
      tails += static_cast<int64_t>(here) * (tmp[i].n_tiles - tmp[i].main_tiles);
    }
    const int split_tiles = static_cast<int>((tails + spare - 1) / spare);
    if (tails > 0 &&
        split_end(tmp, n, split_tiles, tails, head_dim) < 128 * static_cast<int64_t>(tmp[0].n_tiles)) {
      a.item0 = item0;
      a.split_blocks = blocks;
      a.total_tiles = static_cast<int32_t>(tails);
      a.split_tiles = split_tiles;
      a.part_o = split_ws;
      a.part_ml = split_ws + static_cast<size_t>(2) * kAttnSplitBlocks * BQ * head_dim;
      a.per_xcd = blocks / kNumXcd;
      // the full rounds: a whole number of items per XCD
      for (int x = 0; x <= kNumXcd; ++x) a.xcd_begin[x] = item0 / kNumXcd * x;
    } else {
      for (int i = 0; i < n; ++i) tmp[i].main_tiles = tmp[i].n_tiles;
    }
  }
  for (int i = 0; i < n; ++i) a.s[i] = tmp[i];
  if (!a.split_blocks) balance_items_over_xcds(a, false);
}

constexpr size_t kAloneLds = 20 * 1024;   // 64 + 20 KB: one workgroup in a CU's 160 KB
template <int HD, bool P, bool V>
static void launch_attn_t(hipStream_t st, const AttnArgs& a, dim3 grid) {
  if (a.small) {
    hipLaunchKernelGGL((attn_small_kernel<HD, P, V>), grid, dim3(64 * SM_WAVES), 0, st, a);
  } else if (a.split_blocks) {
    if (a.item0 > 0)
      hipLaunchKernelGGL((attn_kernel<HD, P, V>), dim3(a.item0), dim3(NTHR), 0, st, a);
    hipLaunchKernelGGL((attn_split_kernel<HD, P, V>), grid, dim3(NTHR), 0, st, a);
    hipLaunchKernelGGL((attn_merge_kernel<HD>),
                       dim3((a.total_items - a.item0) * (BQ / (256 / (HD / 4)))), dim3(256), 0, st, a);
  } else {
    // (unused LDS that leaves no room for a second workgroup)
    const size_t lds = HD == 64 && a.alone ? kAloneLds : 0;
    hipLaunchKernelGGL((attn_kernel<HD, P, V>), grid, dim3(NTHR), lds, st, a);
  }
}

hipError_t launch_attention(hipStream_t st, const AttnArgs& a, int head_dim, bool paged) {
  if (a.total_items == 0) return hipSuccess;
  const dim3 grid(a.per_xcd * kNumXcd);
  // contiguous keys take the 16-byte value path only when every block length is a multiple of 8
  bool vec = true;
  if (!paged)
    for (int i = 0; i < a.n_streams; ++i) vec = vec && (a.s[i].T % 8 == 0);
  if (head_dim == 128) {
    if (paged) launch_attn_t<128, true, true>(st, a, grid);
    else if (vec) launch_attn_t<128, false, true>(st, a, grid);
    else launch_attn_t<128, false, false>(st, a, grid);
  } else if (head_dim == 64) {
    if (paged) launch_attn_t<64, true, true>(st, a, grid);
    else if (vec) launch_attn_t<64, false, true>(st, a, grid);
    else launch_attn_t<64, false, false>(st, a, grid);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ardit
