// Stage 0, bank indexing (Sec. 3.3.1): subset-seed key of every word, then a
// stable sort by key into CSR form (key_off, occ, occ_seq).
//
// Pass 1's counting kernel also validates the bank against its layout and
// writes the scan codes (the letters scaled to table offsets) that the
// extension kernels read.
//
// The sort is a two-pass LSD radix sort on the 14-bit key: the low 7 bits
// (128 buckets), then the high 7 bits (69 buckets).  Each pass cuts its input
// into tiles of kIxTile elements, one wavefront each, four to a workgroup: a
// counting kernel writes the workgroup's bucket histogram bucket-major, an
// exclusive scan over (bucket, workgroup) gives every workgroup its first slot in
// each bucket, and a scattering kernel ranks each tile's elements in order within
// their bucket (see RankLds) into the tile's own bucket order in LDS, then writes
// the staged tile out bucket by bucket, consecutive lanes on consecutive slots.
// Both passes are stable, so the order inside a key is the position order:
// ascending (sequence, position), independent of scheduling.  Pass 1 reads the
// codes and writes one 64-bit entry per word (position and sequence, from the
// first sequence of the position's tile, which the layout check records per tile)
// and, beside it, the byte of its high digit, which is all that pass 2 ranks by;
// pass 2 writes occ and occ_seq, and key_off follows from the two scanned
// histograms.
//
// 300,000 proteins, some 85M words, between 0.81 GB read and written at least (0.17 ms
// at the rate of a large copy): 0.78 ms, of which pass 2's scattering 0.32, pass
// 1's 0.27 and the counting kernels 0.12; 1.36 ms before ranks came from byte
// tables (scattering 0.50 and 0.49), keys from packed table lookups (counting 0.14)
// and histograms from workgroups (a column a wavefront: 0.10 more in the two
// scans and the gathers of the columns).  The scattering kernels are bound by
// their LDS traffic: half of the accesses fall on random banks.
#include "plast_internal.h"

namespace plast {

namespace {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

constexpr int kIxTile = 2048;                       // elements per tile (32 per lane)
constexpr int kIxWaves = 4;                         // tiles (one per wavefront) per workgroup
constexpr int kIxGroup = kIxTile * kIxWaves;        // elements per histogram column
constexpr int kD0Bits = 7;                          // pass-1 digit: key & 127
constexpr int kD0 = 1 << kD0Bits;
constexpr int kD1 = (kNKeys + kD0 - 1) >> kD0Bits;  // pass-2 digit: key >> 7, 69 values
static_assert(kD1 <= 128, "pass-2 digits must fit 7 bits");

// Keeps the compiler from moving LDS accesses across a step of a wavefront's
// read-then-update of its own LDS table.  The lanes of a wavefront issue LDS
// instructions together and the LDS serves one wavefront's instructions in
// order, so no hardware barrier is needed.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The tile group of a workgroup: workgroups are dealt to the XCDs round robin, and
// each XCD takes runs of kXcdRun consecutive groups.  Neighbouring tiles then write
// their short runs (16 words of a bucket on average, starting anywhere in a line)
// and their histogram columns through one L2.  300,000 proteins 777 us, 864 in
// order; 12M fragments 1854 and 2026; runs of 4 groups 804 and 1885, of 64 785 and
// 1855, and an eighth of the groups each 801 and 2799 (pass 2 has fewer words than
// positions, and the last XCDs none of them).
constexpr unsigned kXcdRun = 16;

__device__ __forceinline__ int64_t xcd_group() {
  constexpr unsigned kPerRun = kMaxQueues * kXcdRun;
  const unsigned base = blockIdx.x / kPerRun * kPerRun, r = blockIdx.x - base;
  if (base + kPerRun > gridDim.x) return blockIdx.x;  // the rest in order
  return base + r % kMaxQueues * kXcdRun + r / kMaxQueues;
}

// Layout check, and the tile table: tile_seq[t] is the sequence holding
// position t * kIxTile (sequence 0 for the leading separators).  A sequence
// writes its tiles only when its own starts are consistent; the table is read
// only when no thread flagged the layout, and then every tile is written.
__device__ __forceinline__ bool layout_bad(const int64_t* __restrict__ seq_start, int64_t i, int32_t n_seqs,
                                           int64_t n_padded, int32_t* __restrict__ tile_seq, int64_t tiles) {
  int64_t s = seq_start[i];
  bool bad = s < kPadLen || s > n_padded;
  if (i == 0 && s != kPadLen) bad = true;
  if (i == n_seqs && s != n_padded) bad = true;
  if (i < n_seqs) {
    const int64_t nx = seq_start[i + 1];
    if (nx - s < kPadLen) bad = true;
    if (!bad) {
      const int64_t lo = i == 0 ? 0 : s;
      for (int64_t t = (lo + kIxTile - 1) / kIxTile; t < tiles && t * kIxTile < nx; ++t) tile_seq[t] = (int32_t)i;
    }
  }
  return bad;
}

// err is cleared before.
__global__ void k_layout_check(const int64_t* __restrict__ seq_start, int32_t n_seqs, int64_t n_padded,
                               int32_t* __restrict__ tile_seq, int64_t tiles, int32_t* __restrict__ err) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n_seqs) return;
  if (layout_bad(seq_start, i, n_seqs, n_padded, tile_seq, tiles)) atomicOr(err, 1);
}

// Up to kLayoutOne sequences, by one workgroup that also clears err: one launch
// instead of two for a query bank.
constexpr int kLayoutThreads = 1024;
constexpr int kLayoutOne = 4 * kLayoutThreads;

__global__ __launch_bounds__(kLayoutThreads) void k_layout_check_one(const int64_t* __restrict__ seq_start,
                                                                     int32_t n_seqs, int64_t n_padded,
                                                                     int32_t* __restrict__ tile_seq, int64_t tiles,
                                                                     int32_t* __restrict__ err) {
  bool bad = false;
  for (int64_t i = threadIdx.x; i <= n_seqs; i += kLayoutThreads)
    bad |= layout_bad(seq_start, i, n_seqs, n_padded, tile_seq, tiles);
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) {
    err[0] = any ? 1 : 0;
    err[1] = 0;
  }
}

// ---------------------------------------------------------------- words of a tile
// A lane works on kPer = 32 consecutive elements of its wavefront's tile, so the
// stable order inside a bucket is (lane, element of the lane).
constexpr int kPer = kIxTile / 64;
static_assert(kPer == 32 && kPadCode < 128, "a lane's residue flags fill one dword; packed compares of codes");

// The kPer + 4 codes from the lane's first position as dwords (separators past n_padded).
__device__ __forceinline__ void lane_codes(const uint8_t* __restrict__ codes, int64_t beg, int64_t n_padded,
                                           uint32_t (&w)[kPer / 4 + 1]) {
  if ((reinterpret_cast<uintptr_t>(codes + beg) & 15) == 0 && beg + kPer + 4 <= n_padded) {
    const uint4 a = *(const uint4*)(codes + beg), b = *(const uint4*)(codes + beg + 16);
    w[0] = a.x, w[1] = a.y, w[2] = a.z, w[3] = a.w;
    w[4] = b.x, w[5] = b.y, w[6] = b.z, w[7] = b.w;
    w[8] = *(const uint32_t*)(codes + beg + kPer);
  } else {
#pragma unroll
    for (int j = 0; j <= kPer / 4; ++j) {
      w[j] = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        w[j] |= (uint32_t)(beg + 4 * j + k < n_padded ? codes[beg + 4 * j + k] : (uint8_t)kPadCode) << (8 * k);
    }
  }
}

// What the words meeting four codes need of them, a byte per code.
struct CodeBytes {
  uint32_t letter;  // the code, 0 where it is no residue
  uint32_t class2;  // class at the seed's second position
  uint32_t class3;  // 20 x class at its third
  uint32_t none;    // 128 where the code is no residue
};

// Bytes of the 20-entry table t at the codes of four bytes; sel, half and top are
// the codes' bits 0-2, 3 and 4 as byte selectors.
__device__ __forceinline__ uint32_t lookup20(const uint32_t (&t)[5], uint32_t sel, uint32_t half, uint32_t top) {
  const uint32_t p0 = __builtin_amdgcn_perm(t[1], t[0], sel), p1 = __builtin_amdgcn_perm(t[3], t[2], sel);
  return __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[4], t[4], sel), __builtin_amdgcn_perm(p1, p0, half), top);
}

// ((w + 108 per byte) | w) has a byte's top bit set iff that byte is >= 20, once
// the carries out of bytes >= 148 are kept from the next byte.
__device__ __forceinline__ uint32_t no_residue(uint32_t w) { return (((w & 0x7F7F7F7Fu) + 0x6C6C6C6Cu) | w) & 0x80808080u; }
__device__ __forceinline__ uint32_t byte_mask(uint32_t top_bits) { return (top_bits << 1) - (top_bits >> 7); }

__device__ __forceinline__ CodeBytes code_bytes(uint32_t w, const SeedClasses& sc) {
  CodeBytes b;
  b.none = no_residue(w);
  b.letter = w & ~byte_mask(b.none);
  const uint32_t sel = b.letter & 0x07070707u;
  const uint32_t half = ((b.letter >> 1) & 0x04040404u) | 0x03020100u;
  const uint32_t top = ((b.letter >> 2) & 0x04040404u) | 0x03020100u;
  b.class2 = lookup20(sc.pos2, sel, half, top);
  b.class3 = lookup20(sc.pos3x20, sel, half, top);
  return b;
}

// Seed keys of the four words starting in lo's bytes (hi: the next four codes), -1
// unless all four codes of the word are residues.  A key is ((2 w0 + class2(w1)) *
// 11 + class3(w2)) * 20 + w3: a byte 2 w0 + class2 <= 39 and a byte 20 class3 + w3
// <= 219, formed for four words at once.
__device__ __forceinline__ void word_keys4(const CodeBytes& lo, const CodeBytes& hi, int (&key)[4]) {
  const uint32_t a = 2 * lo.letter + __builtin_amdgcn_alignbyte(hi.class2, lo.class2, 1);
  const uint32_t b = __builtin_amdgcn_alignbyte(hi.class3, lo.class3, 2) +
                     __builtin_amdgcn_alignbyte(hi.letter, lo.letter, 3);
  const uint32_t none = lo.none | __builtin_amdgcn_alignbyte(hi.none, lo.none, 1) |
                        __builtin_amdgcn_alignbyte(hi.none, lo.none, 2) |
                        __builtin_amdgcn_alignbyte(hi.none, lo.none, 3);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = (int)__umul24((a >> (8 * k)) & 255u, 220u) + (int)((b >> (8 * k)) & 255u);
    key[k] = (none >> (8 * k)) & 128u ? -1 : v;
  }
}

// ---------------------------------------------------------------- ranks in a tile
// Stable ranks within ND buckets, of elements held kPer to a lane.  A table in LDS
// has a byte per (bucket, lane), 16 dwords to a bucket: the element's lane adds 1
// to its byte with a returning atomic on the dword, which gives the element's rank
// among the lane's own (a lane's atomics are served in order, and the other bytes
// of the dword are other lanes'), with no wait between elements.  The bytes of
// each 8 lanes are then replaced by their exclusive prefix sums (at most 7 x 32),
// and a 16-bit entry per (bucket, 8 lanes) gets the first slot of those lanes in
// the tile's bucket order.
// A ballot per digit bit and a running counter per bucket, 64 elements a round,
// took some 60 vector instructions and a dependent LDS read and write a round.
template <int ND>
struct RankLds {
  uint32_t count[ND * 16];
  uint16_t first[ND * 8];
};

template <int ND>
__device__ __forceinline__ void rank_clear(RankLds<ND>& r, int lane) {
  for (int j = lane; j < ND * 4; j += 64) ((uint4*)r.count)[j] = make_uint4(0, 0, 0, 0);
}

template <int ND>
__device__ __forceinline__ uint32_t rank_add(RankLds<ND>& r, int d, bool valid, int lane) {
  const int sh = 8 * (lane & 3);
  return __builtin_amdgcn_ubfe(atomicAdd(&r.count[d * 16 + (lane >> 2)], valid ? 1u << sh : 0u), sh, 8);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, 31
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// Of bucket lane + 64 h: tot[h] its elements in the tile, lst[h] its first slot in
// the tile's bucket order.  Returns the tile's elements.
template <int ND>
__device__ __forceinline__ int rank_scan(RankLds<ND>& r, uint32_t (&tot)[2], uint32_t (&lst)[2], int lane) {
  uint4 v[2][4];
  uint32_t total = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool on = lane + 64 * h < ND;
    tot[h] = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[h][q] = on ? ((const uint4*)(r.count + (lane + 64 * h) * 16))[q] : make_uint4(0, 0, 0, 0);
      tot[h] = __builtin_amdgcn_sad_u8(v[h][q].x, 0, tot[h]);
      tot[h] = __builtin_amdgcn_sad_u8(v[h][q].y, 0, tot[h]);
      tot[h] = __builtin_amdgcn_sad_u8(v[h][q].z, 0, tot[h]);
      tot[h] = __builtin_amdgcn_sad_u8(v[h][q].w, 0, tot[h]);
    }
    const uint32_t incl = wave_incl_scan(tot[h]);
    lst[h] = total + incl - tot[h];
    total += __builtin_amdgcn_readlane(incl, 63);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t run = lst[h], packed[4];
    auto eight = [&](uint32_t& x0, uint32_t& x1) {  // returns the first slot of the eight lanes
      uint32_t t0 = x0 + (x0 << 8), t1 = x1 + (x1 << 8);
      t0 += t0 << 16;
      t1 += t1 << 16;
      const uint32_t first = run;
      run += (t0 >> 24) + (t1 >> 24);
      x1 = t1 - x1 + __builtin_amdgcn_perm(t0, t0, 0x03030303u);
      x0 = t0 - x0;
      return first;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      packed[q] = eight(v[h][q].x, v[h][q].y);
      packed[q] |= eight(v[h][q].z, v[h][q].w) << 16;
    }
    if (lane + 64 * h < ND) {
#pragma unroll
      for (int q = 0; q < 4; ++q) ((uint4*)(r.count + (lane + 64 * h) * 16))[q] = v[h][q];
      *(uint4*)(r.first + (lane + 64 * h) * 8) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
    }
  }
  return (int)total;
}

template <int ND>
__device__ __forceinline__ uint32_t rank_slot(const RankLds<ND>& r, int d, uint32_t own, int lane) {
  return r.first[d * 8 + (lane >> 3)] + ((const uint8_t*)r.count)[d * 64 + lane] + own;
}

// The scanned histogram has a column per workgroup: goff[h] is its first global slot
// in bucket lane + 64 h.  Wavefront wv's tile follows those before it, whose counts
// tot_all holds; delta[d] is what added to a slot of bucket d in the tile's own
// order gives the global slot.  Contains a barrier.
template <int ND>
__device__ __forceinline__ void load_column(const int32_t* __restrict__ offs, int64_t groups, int64_t group,
                                            int32_t (&goff)[2], int lane) {
#pragma unroll
  for (int h = 0; h < 2; ++h) goff[h] = lane + 64 * h < ND ? offs[(int64_t)(lane + 64 * h) * groups + group] : 0;
}

template <int ND>
__device__ __forceinline__ void tile_delta(const int32_t (&goff)[2], const uint32_t (&tot)[2], const uint32_t (&lst)[2],
                                           uint16_t (&tot_all)[kIxWaves][2 * 64], int32_t* delta, int wv, int lane) {
#pragma unroll
  for (int h = 0; h < 2; ++h) tot_all[wv][lane + 64 * h] = (uint16_t)tot[h];
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    int32_t g = goff[h] - (int32_t)lst[h];
#pragma unroll
    for (int k = 0; k < kIxWaves - 1; ++k) g += k < wv ? (int)tot_all[k][lane + 64 * h] : 0;
    if (lane + 64 * h < ND) delta[lane + 64 * h] = g;
  }
  wave_sync();
}

// A workgroup's histogram column from its wavefronts' counts.  Contains a barrier.
template <int ND>
__device__ __forceinline__ void store_column(const int32_t (&cnt)[kIxWaves][kD0], int32_t* __restrict__ hist,
                                             int64_t groups, int64_t group) {
  __syncthreads();
  const int d = threadIdx.x;
  if (d >= ND || group >= groups) return;
  int32_t v = 0;
#pragma unroll
  for (int k = 0; k < kIxWaves; ++k) v += cnt[k][d];
  hist[(int64_t)d * groups + group] = v;
}

// Pass 1, counting, fused with the validation of the bank and the writing of
// the scan codes: one wavefront per tile of kIxTile positions, kPer of them a lane
// (tiles past the bank write the scan codes' tail slack only).  Validation:
// position p is a residue iff some sequence s has seq_start[s] <= p <
// seq_start[s + 1] - kPadLen; residues must be < 20 and every other position
// below n_padded the separator.  The residue positions of the tile come as a
// bitmap, a dword per lane: the state at the tile's first position, toggled at
// every sequence start and every residue end inside the tile (a sequence with no
// residue toggles twice at one position), resolved by a prefix xor within each
// lane's 32 positions and a prefix parity across the lanes.  The scan codes are
// the validated codes times kScale.  The histogram counts the low digit of the key
// of every word starting in the tile, from the raw codes, as the scattering pass
// does: on a valid bank a word of four codes < 20 lies inside one sequence.  After
// a layout error nothing is validated or written but the histogram.
__global__ __launch_bounds__(64 * kIxWaves) void k_ix_check_count1(
    const uint8_t* __restrict__ codes, const int64_t* __restrict__ seq_start, int32_t n_seqs, int64_t n_padded,
    const int32_t* __restrict__ tile_seq, int64_t tiles, uint8_t* __restrict__ scan, int64_t scan_len, SeedClasses sc,
    int32_t* __restrict__ hist, int64_t groups, int32_t* __restrict__ err) {
  __shared__ int32_t cnt_all[kIxWaves][kD0];
  __shared__ uint32_t rb_all[kIxWaves][kIxTile / 32];
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int64_t group = xcd_group(), tile = group * kIxWaves + wv;
  const int64_t beg = tile * kIxTile;
  int32_t* cnt = cnt_all[wv];
  uint32_t* rb = rb_all[wv];
  const int64_t lane_beg = beg + kPer * lane;
  uint32_t w[kPer / 4 + 1];
  lane_codes(codes, lane_beg, n_padded, w);
  cnt[lane] = 0;
  cnt[lane + 64] = 0;
  rb[lane] = 0;
  const bool layout_ok = !(*err & 1);
  wave_sync();
  if (layout_ok) {
    // s0: the last sequence with seq_start <= beg (-1 before the first one)
    int s0 = n_seqs - 1;
    if (beg < n_padded && n_seqs > 0) {
      s0 = min(max(tile_seq[min(tile, tiles - 1)], 0), n_seqs - 1);
      if (seq_start[s0] > beg) s0 = -1;
    }
    const bool init = s0 >= 0 && beg < (s0 + 1 < n_seqs ? seq_start[s0 + 1] : n_padded) - kPadLen;
    // Toggles from the starts s0 + 1 .. s0 + 128 (n_padded standing for
    // seq_start[n_seqs]): a start inside the tile, and the residue end kPadLen
    // before it.  A valid layout puts at most 104 of them within kIxTile + kPadLen
    // of beg, since consecutive starts are at least kPadLen apart.
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t idx = (int64_t)s0 + 1 + k * 64 + lane;
      if (idx <= n_seqs) {
        const int64_t v = idx < n_seqs ? seq_start[idx] : n_padded;
        const int64_t e = v - kPadLen;
        if (idx < n_seqs && v > beg && v < beg + kIxTile) atomicXor(&rb[(v - beg) >> 5], 1u << ((v - beg) & 31));
        if (e > beg && e < beg + kIxTile) atomicXor(&rb[(e - beg) >> 5], 1u << ((e - beg) & 31));
      }
    }
    wave_sync();
    const uint32_t tog = rb[lane];
    uint32_t x = tog;
    x ^= x << 1;
    x ^= x << 2;
    x ^= x << 4;
    x ^= x << 8;
    x ^= x << 16;
    const uint64_t odd = __ballot(__popc(tog) & 1);
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const bool flip = ((__popcll(odd & below) & 1) != 0) != init;
    const uint32_t residues = flip ? ~x : x;
    uint32_t bad = 0, out[kPer / 4];
#pragma unroll
    for (int j = 0; j < kPer / 4; ++j) {
      // the four flags as byte masks
      const uint32_t res = byte_mask((__umul24((residues >> (4 * j)) & 15u, 0x204081u) << 7) & 0x80808080u);
      const uint32_t none = no_residue(w[j]);
      bad |= ((w[j] ^ (0x01010101u * kPadCode)) & ~res) | (none & res);
      const uint32_t keep = res & ~byte_mask(none);
      out[j] = ((w[j] & keep) | ((0x01010101u * kPadCode) & ~keep)) * kScale;
    }
    // scan is 256-byte aligned and scan_len a multiple of 256
    if (lane_beg < scan_len) {
      uint4* dst = (uint4*)(scan + lane_beg);
      dst[0] = make_uint4(out[0], out[1], out[2], out[3]);
      dst[1] = make_uint4(out[4], out[5], out[6], out[7]);
    }
    if (__ballot(bad != 0) != 0 && lane == 0) atomicOr(err, 2);
  }
  CodeBytes lo = code_bytes(w[0], sc);
#pragma unroll
  for (int j = 0; j < kPer / 4; ++j) {
    const CodeBytes hi = code_bytes(w[j + 1], sc);
    int key[4];
    word_keys4(lo, hi, key);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (key[k] >= 0) atomicAdd(&cnt[key[k] & (kD0 - 1)], 1);
    lo = hi;
  }
  store_column<kD0>(cnt_all, hist, groups, group);
}

// Pass 1, scattering: the tile's words, ranked within their low digit, are put in
// the tile's own bucket order in LDS (key | position offset << 14 | sequence offset
// << 25) and written out from there bucket by bucket, consecutive lanes to
// consecutive slots: the position and sequence as one 64-bit entry, the high digit
// beside it.  Runs only on a valid layout (the tile table is complete, a tile meets
// at most 103 sequence starts and the words fit the word array).
// 300,000 proteins, some 85M words: 272 us, 490 us when ranked by ballots (75% of the
// vector issue rate).
static_assert(kIxTile == 2048, "word staging packs a position offset in 11 bits");

__global__ __launch_bounds__(64 * kIxWaves) void k_ix_scatter1(
    const uint8_t* __restrict__ codes, const int64_t* __restrict__ seq_start, int32_t n_seqs, int64_t n_padded,
    int64_t tiles, int64_t groups, SeedClasses sc, const int32_t* __restrict__ tile_seq,
    const int32_t* __restrict__ err, const int32_t* __restrict__ offs, int64_t cap, uint2* __restrict__ words, uint8_t* __restrict__ digits) {
  union Lds {  // the ranks' table is read before the stage is written
    RankLds<kD0> rank;
    uint32_t stage[kIxTile];
  };
  __shared__ __align__(16) Lds lds_all[kIxWaves];
  __shared__ int32_t delta_all[kIxWaves][kD0];
  __shared__ uint32_t sbits_all[kIxWaves][64];
  __shared__ uint16_t tot_all[kIxWaves][2 * 64];
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int64_t group = xcd_group(), tile = group * kIxWaves + wv;
  if (n_seqs == 0 || (*err & 1)) return;  // (a tile past the last holds no word)
  RankLds<kD0>& rank = lds_all[wv].rank;
  uint32_t* stage = lds_all[wv].stage;
  int32_t* delta = delta_all[wv];
  uint32_t* sbits = sbits_all[wv];
  const int64_t beg = tile * kIxTile;
  uint32_t w[kPer / 4 + 1];
  lane_codes(codes, beg + kPer * lane, n_padded, w);
  int32_t goff[2];
  load_column<kD0>(offs, groups, group, goff, lane);
  const int s0 = min(max(tile_seq[min(tile, tiles - 1)], 0), n_seqs - 1);
  // The sequence starts s0 + 1 .. s0 + 128 inside the tile as a bitmap, a dword per
  // lane: a position's sequence is s0 + the starts at or before it.
  sbits[lane] = 0;
  rank_clear(rank, lane);
  wave_sync();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int64_t idx = (int64_t)s0 + 1 + k * 64 + lane;
    const int64_t o = (idx < n_seqs ? seq_start[idx] : INT64_MAX) - beg;
    if (o > 0 && o < kIxTile) atomicOr(&sbits[o >> 5], 1u << (o & 31));
  }
  wave_sync();
  const uint32_t starts = sbits[lane];
  int seq = (int)wave_incl_scan(__popc(starts)) - __popc(starts);
  uint32_t e[kPer], own[kPer];
  {
    CodeBytes lo = code_bytes(w[0], sc);
#pragma unroll
    for (int j = 0; j < kPer / 4; ++j) {
      const CodeBytes hi = code_bytes(w[j + 1], sc);
      int key[4];
      word_keys4(lo, hi, key);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = 4 * j + k;
        seq += (int)((starts >> i) & 1u);
        own[i] = rank_add(rank, key[k] & (kD0 - 1), key[k] >= 0, lane);
        e[i] = key[k] < 0 ? ~0u  // no key is 16383
                          : (uint32_t)key[k] | ((uint32_t)(kPer * lane + i) << 14) | ((uint32_t)min(seq, 127) << 25);
      }
      lo = hi;
    }
  }
  wave_sync();
  uint32_t tot[2], lst[2];
  const int nt = rank_scan(rank, tot, lst, lane);
  wave_sync();
#pragma unroll
  for (int i = 0; i < kPer; ++i) own[i] = rank_slot(rank, (int)(e[i] & (kD0 - 1)), own[i], lane);
  wave_sync();
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (e[i] != ~0u && own[i] < (uint32_t)kIxTile) stage[own[i]] = e[i];
  tile_delta<kD0>(goff, tot, lst, tot_all, delta, wv, lane);
#pragma unroll 4
  for (int l = lane; l < min(nt, kIxTile); l += 64) {
    const uint32_t v = stage[l];
    const int key = (int)(v & 0x3fffu);
    const int64_t slot = (int64_t)delta[key & (kD0 - 1)] + l;
    if (slot >= 0 && slot < cap) {
      words[slot] = make_uint2((uint32_t)beg + ((v >> 14) & 2047u), (uint32_t)s0 + (v >> 25));
      digits[slot] = (uint8_t)min(key >> kD0Bits, kD1 - 1);
    }
  }
}

// Pass 2, counting: histogram of the high digit over the words of a workgroup's
// tiles, read from the byte per word that pass 1 writes beside each entry (the array
// is 256-byte aligned and padded, so 16 bytes that straddle the end stay inside it).
__global__ __launch_bounds__(64 * kIxWaves) void k_ix_count2(const uint8_t* __restrict__ digits,
                                                            const int32_t* __restrict__ err, int64_t cap,
                                                            int64_t groups, int32_t* __restrict__ hist) {
  __shared__ int32_t cnt_all[kIxWaves][kD0];
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int64_t group = xcd_group();
  if (*err & 1) return;
  int32_t* cnt = cnt_all[wv];
  cnt[lane] = 0;
  cnt[lane + 64] = 0;
  wave_sync();
  const int64_t n = min((int64_t)err[1], cap);
  const int64_t beg = group * kIxGroup + wv * kIxTile;
#pragma unroll
  for (int r = 0; r < kIxTile / 1024; ++r) {
    const int64_t i = beg + r * 1024 + 16 * lane;
    if (i < n) {
      const uint4 v = *(const uint4*)(digits + i);
      const uint32_t d4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (i + k < n) atomicAdd(&cnt[min((int)((d4[k >> 2] >> (8 * (k & 3))) & 0xffu), kD1 - 1)], 1);
    }
  }
  store_column<kD1>(cnt_all, hist, groups, group);
}

// Pass 2, scattering: a lane ranks the words of its 32 digits; the slots go back
// through LDS to the lanes that read the words, consecutive lanes consecutive
// words, which put them in the tile's bucket order in LDS, to be written out as occ
// and occ_seq.  Some 85M words: 317 us, 499 us when ranked by ballots; positions and
// sequences staged one after the other in half the LDS: 395 us.
__global__ __launch_bounds__(64 * kIxWaves) void k_ix_scatter2(const uint2* __restrict__ words,
                                                               const uint8_t* __restrict__ digits,
                                                               const int32_t* __restrict__ err, int64_t cap,
                                                               int64_t groups, const int32_t* __restrict__ offs,
                                                               int32_t* __restrict__ occ,
                                                               int32_t* __restrict__ occ_seq) {
  union Lds {  // each is read before the next one is written
    RankLds<kD1> rank;
    uint16_t slot[kIxTile];
    uint2 stage[kIxTile];
  };
  __shared__ __align__(16) Lds lds_all[kIxWaves];
  __shared__ uint8_t dig_all[kIxWaves][kIxTile];  // digits in bucket order
  __shared__ int32_t delta_all[kIxWaves][kD1];
  __shared__ uint16_t tot_all[kIxWaves][2 * 64];
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  const int64_t group = xcd_group();
  RankLds<kD1>& rank = lds_all[wv].rank;
  uint2* stage = lds_all[wv].stage;
  uint8_t* dig = dig_all[wv];
  int32_t* delta = delta_all[wv];
  const int64_t n = min((int64_t)err[1], cap);
  if ((*err & 1) || group * kIxGroup >= n) return;
  const int64_t beg = group * kIxGroup + wv * kIxTile;
  const int nw = (int)max(min((int64_t)kIxTile, n - beg), (int64_t)0);  // the tile's words
  int32_t goff[2];
  load_column<kD1>(offs, groups, group, goff, lane);
  // Elements past the last word take the last digit and so the slots past it.
  const int mine = nw - kPer * lane;  // words of the lane
  uint32_t d4[kPer / 4];
  {
    uint4 a = make_uint4(~0u, ~0u, ~0u, ~0u), b = a;
    if (mine > 0) {  // the array's end is a multiple of 256 past its start
      a = *(const uint4*)(digits + beg + kPer * lane);
      b = *(const uint4*)(digits + beg + kPer * lane + 16);
    }
    d4[0] = a.x, d4[1] = a.y, d4[2] = a.z, d4[3] = a.w;
    d4[4] = b.x, d4[5] = b.y, d4[6] = b.z, d4[7] = b.w;
  }
  uint2 e[kPer];
  if (nw == kIxTile) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) e[i] = words[beg + i * 64 + lane];
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) e[i] = words[min(beg + i * 64 + lane, n - 1)];
#pragma unroll
    for (int j = 0; j < kPer / 4; ++j) {
      const int past = min(max(4 * (j + 1) - mine, 0), 4);  // bytes of the dword past the last word
      d4[j] |= past ? ~0u << (32 - 8 * past) : 0u;
    }
  }
  rank_clear(rank, lane);
  wave_sync();
  auto digit = [&](int i) { return min((int)__builtin_amdgcn_ubfe(d4[i >> 2], 8 * (i & 3), 8), kD1 - 1); };
  uint32_t slot[kPer / 2];  // 16 bits each
  {
    uint32_t own[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) own[i] = rank_add(rank, digit(i), true, lane);
    wave_sync();
    uint32_t tot[2], lst[2];
    rank_scan(rank, tot, lst, lane);
    const int past = kIxTile - nw;  // elements past the last word, counted with the last digit
    if (lane == (kD1 - 1) % 64) tot[(kD1 - 1) / 64] -= past;
    tile_delta<kD1>(goff, tot, lst, tot_all, delta, wv, lane);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t at = min(rank_slot(rank, digit(i), own[i], lane), (uint32_t)kIxTile - 1);
      dig[at] = (uint8_t)digit(i);
      slot[i / 2] = i & 1 ? slot[i / 2] | (at << 16) : at;
    }
  }
  wave_sync();
  uint4* dst = (uint4*)(lds_all[wv].slot + kPer * lane);
#pragma unroll
  for (int q = 0; q < kPer / 8; ++q)
    dst[q] = make_uint4(slot[4 * q], slot[4 * q + 1], slot[4 * q + 2], slot[4 * q + 3]);
  wave_sync();
#pragma unroll
  for (int i = 0; i < kPer; i += 2)
    slot[i / 2] = lds_all[wv].slot[i * 64 + lane] | ((uint32_t)lds_all[wv].slot[i * 64 + 64 + lane] << 16);
  auto slot_of = [&](int i) { return (slot[i / 2] >> (16 * (i & 1))) & 0xffffu; };
  wave_sync();
#pragma unroll
  for (int i = 0; i < kPer; ++i) stage[slot_of(i)] = e[i];
  wave_sync();
#pragma unroll 8
  for (int l = lane; l < nw; l += 64) {
    const uint2 v = stage[l];
    const int g = delta[min((int)dig[l], kD1 - 1)] + l;
    if ((unsigned)g < (unsigned)n) {
      occ[g] = (int32_t)v.x;
      occ_seq[g] = (int32_t)v.y;
    }
  }
}

__global__ void k_clear2(int32_t* __restrict__ p) {
  if (threadIdx.x < 2) p[threadIdx.x] = 0;
}

// key_off from the two scanned histograms, with no pass over the sorted words.
// After pass 1 the word array is ordered by the low digit: the words whose low
// digit is below lo are its first offs1[lo * groups1] entries.  Pass 2 cuts that
// array into groups of kIxGroup entries, and its scanned histogram holds, for
// high digit d and group t, the words of high digit below d plus those of high
// digit d in the groups before t.  So the words with key below k = d * 128 + lo
// number offs2[d * groups2 + t] for the group t holding entry offs1[lo * groups1],
// plus the words of high digit d in that group before the entry, which one
// workgroup per low digit counts (fewer than kIxGroup entries).  A key with no
// word gets the first slot of the next key that has one, n_words past the
// last.  After a layout error the index holds no word.
__global__ __launch_bounds__(256) void k_ix_key_off(const uint8_t* __restrict__ digits,
                                                    const int32_t* __restrict__ offs1, int64_t groups1,
                                                    const int32_t* __restrict__ offs2, int64_t groups2,
                                                    const int32_t* __restrict__ err, int64_t cap,
                                                    int64_t* __restrict__ key_off) {
  __shared__ int32_t cnt[kD1];
  const int lo = blockIdx.x;
  const bool none = (err[0] & 1) != 0;
  const int64_t n = none ? 0 : min((int64_t)err[1], cap);
  for (int d = threadIdx.x; d < kD1; d += blockDim.x) cnt[d] = 0;
  __syncthreads();
  const int64_t start = none ? 0 : min(max((int64_t)offs1[(int64_t)lo * groups1], (int64_t)0), n);
  const int64_t t = start / kIxGroup;
  for (int64_t i = t * kIxGroup + 16 * threadIdx.x; i < start; i += 16 * blockDim.x) {
    const uint4 v = *(const uint4*)(digits + i);  // (the array's end is a multiple of 256 past its start)
    const uint32_t d4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (i + k < start) atomicAdd(&cnt[min((int)((d4[k >> 2] >> (8 * (k & 3))) & 0xffu), kD1 - 1)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < kD1; d += blockDim.x) {
    const int k = d * kD0 + lo;
    if (k >= kNKeys) continue;
    int64_t v = 0;
    if (!none) {
      const int64_t idx = (int64_t)d * groups2 + t;
      v = min((idx < (int64_t)kD1 * groups2 ? (int64_t)offs2[idx] : n) + cnt[d], n);
    }
    key_off[k] = v;
  }
  if (lo == 0 && threadIdx.x == 0) key_off[kNKeys] = n;
}

// ---------------------------------------------------------------- scan
// Exclusive scans in place, in as few launches as the length allows (a launch costs
// about 5 us where little else runs): one workgroup up to kScanOne elements; up to
// kScanTops blocks, a local scan of each block and then one pass in which every
// block sums the totals before its own (8 KB of L2 reads a block on average at
// most); beyond, where those reads would exceed the data, a scan of the totals in
// between.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanBlock = kScanThreads * kScanPer;
constexpr int kScanTops = 4096;
constexpr int kScanOneThreads = 1024;
constexpr int kScanOnePer = 16;
constexpr int kScanOne = kScanOneThreads * kScanOnePer;

// Workgroup-wide exclusive scan of one value per thread (contains barriers).
template <int NT>
__device__ __forceinline__ int block_excl_scan(int v, int* total) {
  __shared__ int wsum[NT / 64];
  int lane = lane_id(), wid = threadIdx.x / 64;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    before += (w < wid) ? wsum[w] : 0;
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

// PER consecutive elements from `base` (0 past n), 16 bytes at a time where they
// all exist; data is 16-byte aligned and base a multiple of 4.
template <int PER>
__device__ __forceinline__ void load_run(const int32_t* __restrict__ data, int64_t base, int64_t n, int (&v)[PER]) {
  if (base + PER <= n) {
#pragma unroll
    for (int i = 0; i < PER; i += 4) {
      const int4 x = *(const int4*)(data + base + i);
      v[i] = x.x;
      v[i + 1] = x.y;
      v[i + 2] = x.z;
      v[i + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = base + i < n ? data[base + i] : 0;
  }
}

template <int PER>
__device__ __forceinline__ void store_run(int32_t* __restrict__ data, int64_t base, int64_t n, const int (&v)[PER]) {
  if (base + PER <= n) {
#pragma unroll
    for (int i = 0; i < PER; i += 4) *(int4*)(data + base + i) = make_int4(v[i], v[i + 1], v[i + 2], v[i + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (base + i < n) data[base + i] = v[i];
  }
}

// One block: the exclusive scan of its elements in place; returns their sum.
template <int NT, int PER>
__device__ __forceinline__ int scan_block(int32_t* __restrict__ data, int64_t base, int64_t n) {
  int v[PER], sum = 0;
  load_run<PER>(data, base, n, v);
#pragma unroll
  for (int i = 0; i < PER; ++i) sum += v[i];
  int total;
  int run = block_excl_scan<NT>(sum, &total);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int x = v[i];
    v[i] = run;
    run += x;
  }
  store_run<PER>(data, base, n, v);
  return total;
}

__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(int32_t* __restrict__ data, int64_t n,
                                                              int32_t* __restrict__ grand) {
  const int total = scan_block<kScanOneThreads, kScanOnePer>(data, (int64_t)threadIdx.x * kScanOnePer, n);
  if (threadIdx.x == 0 && grand) *grand = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_local(int32_t* __restrict__ data, int64_t n,
                                                             int32_t* __restrict__ tops) {
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
  const int total = scan_block<kScanThreads, kScanPer>(data, base, n);
  if (threadIdx.x == 0) tops[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_tops(int32_t* __restrict__ tops, int64_t nb,
                                                            int32_t* __restrict__ grand) {
  int carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kScanBlock) {
    int64_t base = b0 + (int64_t)threadIdx.x * kScanPer;
    int v[kScanPer];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
      v[i] = (base + i < nb) ? tops[base + i] : 0;
      sum += v[i];
    }
    int total;
    int run = carry + block_excl_scan<kScanThreads>(sum, &total);
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
      if (base + i < nb) tops[base + i] = run;
      run += v[i];
    }
    carry += total;
  }
  if (threadIdx.x == 0 && grand) *grand = carry;
}

// SCANNED: tops hold the exclusive scan of the blocks' totals; otherwise the
// totals themselves, which the block sums up to its own.
template <bool SCANNED>
__global__ __launch_bounds__(kScanThreads) void k_scan_add(int32_t* __restrict__ data, int64_t n,
                                                           const int32_t* __restrict__ tops,
                                                           int32_t* __restrict__ grand) {
  int add = 0;
  if (SCANNED) {
    add = tops[blockIdx.x];
  } else {
    __shared__ int wsum[kScanThreads / 64];
    int v = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) v += tops[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane_id() == 0) wsum[threadIdx.x / 64] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) add += wsum[w];
    if (threadIdx.x == 0 && grand && blockIdx.x == gridDim.x - 1) *grand = add + tops[blockIdx.x];
  }
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
  int v[kScanPer];
  load_run<kScanPer>(data, base, n, v);
#pragma unroll
  for (int i = 0; i < kScanPer; ++i) v[i] += add;
  store_run<kScanPer>(data, base, n, v);
}

}  // namespace

size_t scan_tmp_bytes(int64_t n) { return align_up(sizeof(int32_t) * (size_t)((n + kScanBlock - 1) / kScanBlock + 1), 256); }

void exclusive_scan_i32(int32_t* d_data, int64_t n, int32_t* d_total, void* d_tmp, hipStream_t s) {
  if (n <= kScanOne) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneThreads), 0, s, d_data, n, d_total);
    return;
  }
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  int32_t* tops = (int32_t*)d_tmp;
  hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(kScanThreads), 0, s, d_data, n, tops);
  if (nb <= kScanTops) {
    hipLaunchKernelGGL(k_scan_add<false>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, d_data, n,
                       (const int32_t*)tops, d_total);
    return;
  }
  hipLaunchKernelGGL(k_scan_tops, dim3(1), dim3(kScanThreads), 0, s, tops, nb, d_total);
  hipLaunchKernelGGL(k_scan_add<true>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, d_data, n, (const int32_t*)tops,
                     (int32_t*)nullptr);
}

IndexLayout index_layout(int64_t n_padded) {
  IndexLayout L;
  size_t off = 0;
  L.key_off = off;
  off = align_up(off + sizeof(int64_t) * (kNKeys + 1), 256);
  L.occ = off;
  off = align_up(off + sizeof(int32_t) * (size_t)n_padded, 256);
  L.occ_seq = off;
  off = align_up(off + sizeof(int32_t) * (size_t)n_padded, 256);
  L.scan = off;
  off = align_up(off + (size_t)n_padded + kScanSlack, 256);
  L.total = off;
  return L;
}

// Workspace: [error words (256 B)] [tile table] [pass-1 histogram] [pass-2 histogram]
// [scan scratch] [word entries between the passes (64-bit)] [their high digits (8-bit)].
// The word arrays hold n_padded - kPadLen entries, a bound on the residues of any valid
// layout that grows with n_padded alone, so a workspace sized for the largest
// bank serves every smaller one whatever its number of sequences.
struct IxWs {
  int64_t tiles1, groups1, groups2, cap;
  size_t tile_seq, hist1, hist2, tmp, words, digits, total;
};

IxWs ix_ws(int64_t n_padded) {
  IxWs w;
  w.cap = n_padded > kPadLen ? n_padded - kPadLen : 0;
  w.tiles1 = (n_padded + kIxTile - 1) / kIxTile;
  if (w.tiles1 < 1) w.tiles1 = 1;
  w.groups1 = (w.tiles1 + kIxWaves - 1) / kIxWaves;
  w.groups2 = (w.cap + kIxGroup - 1) / kIxGroup;
  if (w.groups2 < 1) w.groups2 = 1;
  size_t off = 256;
  w.tile_seq = off;
  off = align_up(off + sizeof(int32_t) * (size_t)w.tiles1, 256);
  w.hist1 = off;
  off = align_up(off + sizeof(int32_t) * (size_t)(kD0 * w.groups1), 256);
  w.hist2 = off;
  off = align_up(off + sizeof(int32_t) * (size_t)(kD1 * w.groups2), 256);
  w.tmp = off;
  const int64_t scan_n = kD0 * w.groups1 > kD1 * w.groups2 ? kD0 * w.groups1 : kD1 * w.groups2;
  off = align_up(off + scan_tmp_bytes(scan_n), 256);
  w.words = off;
  off = align_up(off + sizeof(uint64_t) * (size_t)w.cap, 256);
  w.digits = off;
  off = align_up(off + (size_t)w.cap, 256);
  w.total = off;
  return w;
}

size_t index_ws_bytes(int64_t n_padded) { return ix_ws(n_padded).total; }

int index_enqueue(const uint8_t* d_codes, const int64_t* d_seq_start, int32_t n_seqs, int64_t n_padded,
                  void* d_index, void* d_ws, int32_t* d_err, plast_index_t* out, hipStream_t stream) {
  IndexLayout L = index_layout(n_padded);
  const IxWs W = ix_ws(n_padded);
  uint8_t* base = (uint8_t*)d_index;
  int64_t* key_off = (int64_t*)(base + L.key_off);
  int32_t* occ = (int32_t*)(base + L.occ);
  int32_t* occ_seq = (int32_t*)(base + L.occ_seq);
  uint8_t* scan = base + L.scan;
  int64_t scan_len = (int64_t)(L.total - L.scan);

  uint8_t* ws = (uint8_t*)d_ws;
  int32_t* total = d_err + 1;
  int32_t* tile_seq = (int32_t*)(ws + W.tile_seq);
  int32_t* hist1 = (int32_t*)(ws + W.hist1);
  int32_t* hist2 = (int32_t*)(ws + W.hist2);
  void* tmp = ws + W.tmp;
  uint2* words = (uint2*)(ws + W.words);
  uint8_t* digits = ws + W.digits;

  SeedClasses sc = seed_classes();
  timing_mark(kStageIndex, false, stream);
  if (n_seqs < kLayoutOne) {
    hipLaunchKernelGGL(k_layout_check_one, dim3(1), dim3(kLayoutThreads), 0, stream, d_seq_start, n_seqs, n_padded,
                       tile_seq, W.tiles1, d_err);
  } else {
    // a fill kernel rather than a memset node, so that the sequence can be captured in a graph
    hipLaunchKernelGGL(k_clear2, dim3(1), dim3(64), 0, stream, d_err);
    hipLaunchKernelGGL(k_layout_check, dim3((unsigned)((n_seqs + 1 + 255) / 256)), dim3(256), 0, stream, d_seq_start,
                       n_seqs, n_padded, tile_seq, W.tiles1, d_err);
  }
  // After a layout error the passes that read the tile table or the word
  // arrays return at once and key_off says the index holds no word.
  const unsigned g1 = (unsigned)W.groups1, g2 = (unsigned)W.groups2;
  const int64_t groups_scan = (scan_len + kIxGroup - 1) / kIxGroup;  // covering the scan codes and their slack
  const unsigned gc = (unsigned)(groups_scan > W.groups1 ? groups_scan : W.groups1);
  const dim3 block(64 * kIxWaves);
  hipLaunchKernelGGL(k_ix_check_count1, dim3(gc), block, 0, stream, d_codes, d_seq_start, n_seqs, n_padded,
                     (const int32_t*)tile_seq, W.tiles1, scan, scan_len, sc, hist1, W.groups1, d_err);
  exclusive_scan_i32(hist1, kD0 * W.groups1, total, tmp, stream);
  hipLaunchKernelGGL(k_ix_scatter1, dim3(g1), block, 0, stream, d_codes, d_seq_start, n_seqs, n_padded, W.tiles1,
                     W.groups1, sc, (const int32_t*)tile_seq, (const int32_t*)d_err, (const int32_t*)hist1, W.cap, words,
                     digits);
  hipLaunchKernelGGL(k_ix_count2, dim3(g2), block, 0, stream, (const uint8_t*)digits, (const int32_t*)d_err, W.cap,
                     W.groups2, hist2);
  exclusive_scan_i32(hist2, kD1 * W.groups2, nullptr, tmp, stream);
  hipLaunchKernelGGL(k_ix_scatter2, dim3(g2), block, 0, stream, (const uint2*)words, (const uint8_t*)digits,
                     (const int32_t*)d_err, W.cap, W.groups2, (const int32_t*)hist2, occ, occ_seq);
  hipLaunchKernelGGL(k_ix_key_off, dim3(kD0), dim3(256), 0, stream, (const uint8_t*)digits, (const int32_t*)hist1,
                     W.groups1, (const int32_t*)hist2, W.groups2, (const int32_t*)d_err, W.cap, key_off);
  timing_mark(kStageIndex, true, stream);
  PLAST_HIP(hipGetLastError());

  out->codes = d_codes;
  out->seq_start = d_seq_start;
  out->n_seqs = n_seqs;
  out->n_padded = n_padded;
  out->key_off = key_off;
  out->occ = occ;
  out->occ_seq = occ_seq;
  out->scan_codes = scan;
  out->n_words = -1;
  return PLAST_OK;
}

int build_index_impl(const uint8_t* d_codes, const int64_t* d_seq_start, int32_t n_seqs, int64_t n_padded,
                     void* d_index, void* d_ws, plast_index_t* out, hipStream_t stream) {
  int32_t* err = (int32_t*)d_ws;  // [0] error bits, [1] word total
  plast_index_t view;
  int rc = index_enqueue(d_codes, d_seq_start, n_seqs, n_padded, d_index, d_ws, err, &view, stream);
  if (rc != PLAST_OK) return rc;
  int32_t h_err[2] = {0, 0};
  PLAST_HIP(hipMemcpyAsync(h_err, err, sizeof(h_err), hipMemcpyDeviceToHost, stream));
  PLAST_HIP(hipStreamSynchronize(stream));
  if (h_err[0] & 1) return set_error(PLAST_E_LAYOUT, "seq_start does not describe the padded layout");
  if (h_err[0] & 2) return set_error(PLAST_E_ALPHABET, "a residue code is > 19 or a separator code is not 20");
  view.n_words = h_err[1];
  *out = view;
  return PLAST_OK;
}

}  // namespace plast
