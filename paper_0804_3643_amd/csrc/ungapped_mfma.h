// The ungapped extension on the matrix cores (included by ungapped.hip, inside
// its namespace).
//
// A prefix sum of substitution scores is a contraction: with the bank-b letters
// as one-hot vectors and the bank-a letters as rows of the matrix, step t of all
// pairs of a 32 x 32 tile is a rank-20 product, and the accumulators of a chain
// of MFMAs hold the running prefix sums.  One v_mfma_f32_32x32x64_f8f6f4 has
// room for three letters (60 of its 64 k slots), and two steps fit in one
// MFMA with one maximum: with s = s+ + s- (positive and negative part), the
// chain
//   C(k) = C(k-1) + s-(2k-1) + s(2k) + s+(2k+1)
// gives C(k) = P(2k) + s+(2k+1) = max(P(2k), P(2k+1)), P(t) being the prefix sum
// through step t, so the best prefix is the maximum of 0 and the C(k): 12 MFMAs for
// the 24 rightward steps, then 10 for the leftward ones, whose chain starts
// from the best of the right side (the composition of the VALU tile).  Two
// C(k) enter one v_max3_f32, 8 a lane per MFMA, which is what bounds the
// kernel: an MFMA takes 33 to 37 cycles of a SIMD by itself, with 8 v_max3_f32 of
// unrelated registers 43, and with the accumulators of the step before kept for its
// maxima, as here, 47 (measured with nothing else in the loop, 2 wavefronts per SIMD):
// 24 a step, where the VALU tile needs 60.
//
// Exactness.  The profile holds score / 2 in 6 bits (E2M3, multiples of 1/2 up
// to 7.5: every integer score up to 15 in magnitude, kMaxEntry; other matrices
// take the VALU tile), the one-hot 2.0 in 4 bits (E2M1), the accumulators are
// float: every partial sum is an integer below 2^24.
//
// A bank-b separator is the zero vector: it adds 0 where the VALU tile adds
// kSepScore <= 0.  Both leave the best prefix alone, since a scan that has left
// its sequence meets separators only.  A bank-a separator scores kSepScore.
//
// Layout.  The lane l of an operand holds row (or column) l & 31 and the k slots
// 32 (l >> 5) .. + 31.  Slots 0..19 of the lower half are the letters of step
// 2k, of the upper half those of step 2k + 1 (s+); slots 20..29 are the letters
// 0..9 (lower half) and 10..19 (upper half) of step 2k - 1 (s-).  The rows of an
// item (two tiles of 32) are laid out in LDS once (33.8 KB a tile) and read by
// every wavefront in order, 24 bytes a lane per MFMA; a wavefront builds the one-hot
// operands of 32 columns from two 168-byte tables in LDS, without bank conflicts, one
// side at a time (48 registers, then 40), and uses them for both tiles.  78 KB per
// workgroup of 4 wavefronts: two workgroups on a compute unit, so that one works while
// the other builds its profile.
//
// Measured: 10,000 x 100,000 proteins (1.65e10 pairs) 12.8 ms, 19.2 on the VALU tile
// alone; 1,001 proteins against 1.5M fragments 1.25 and 1.81 ms.  A tile takes about
// 1950 cycles of a SIMD: 1050 for the MFMAs and maxima, the rest for the one-hot
// operands of its columns, its hits, and the item's profile and end.  With few
// rows a key and a bank b that no cache holds, the windows are the bound as well: 450
// proteins against 1M read 60 GB of lines in 10.9 ms.
constexpr int kMThreads = 256;
constexpr int kMWaves = kMThreads / 64;
constexpr int kMTile = 32;
constexpr int kMRows = 2 * kMTile;            // rows of a work item
constexpr int kMSteps = kSpan / 2;            // MFMAs of a tile (22)
constexpr int kMRight = kRight / 2;           // of which rightward (12)
constexpr int kMaxEntry = 15;                 // |score| that E2M3 holds at half its value
constexpr int kMAhead = 4;                    // profile operands in flight
constexpr int kMSlots = 256;                  // staged hits of a wavefront
// Hits are counted before they are written where the staging area has filled, a
// wavefront's groups of 32 columns have had kMHotHits on average and more than kMHotRest
// of them are left (1000 x 30,000 proteins at thresholds of 30 and 25: 869 and 1418 us;
// from 48 hits on 914 and 1542, from 160 on 870 and 1507).
constexpr int kMHotHits = 96, kMHotRest = 2;
static_assert(kRight % 2 == 0 && kNbr % 2 == 0 && kMRight % 2 == 0 && kMSteps % 2 == 0, "two steps per MFMA, two MFMAs per maximum");
static_assert(kMSlots >= 4 * 64, "staged hits: four registers of a tile");
static_assert(kMaxItemCols <= 1 << 14 && kMRows <= 1 << 6 && kSpan * kMaxEntry < 1 << 10, "a staged hit packs row, score and column in 30 bits");

typedef int mi8 __attribute__((ext_vector_type(8)));
typedef float mf16 __attribute__((ext_vector_type(16)));
typedef uint32_t mu2 __attribute__((ext_vector_type(2)));
typedef uint32_t mu4 __attribute__((ext_vector_type(4)));

// An item of kMNarrow rows at most (the rest of a key, or a key of a small query
// bank) takes the VALU tile, whose cost goes with its 4-row groups (about 330
// cycles of a SIMD each per 32 x 32 pairs' columns), while a tile here costs about
// 1950 for any rows.  A 3-protein query against
// 100,000 proteins: 0.21 ms without the rule, 0.14 with it; 450 proteins against 1M:
// 12.3 and 11.6 ms (limits of 8, 12 and 16 rows within 1%).
constexpr int kMNarrow = 8;
static_assert(kMNarrow == 8, "run_narrow has tiles of 4 and 8 rows");

struct __align__(16) MSmem {
  uint2 hot[2][kNLet];             // one-hot of a letter in slots 0..19: dwords 0, 1 and 2, 3 (LDS offset 0)
  uint2 part[2][kNLet];            // one-hot in slots 20..29 (dwords 2, 3), by half
  union {
    struct {
      mu4 a4[2][kMSteps][64];      // profile operands, dwords 0..3 and
      mu2 a2[2][kMSteps][64];      // 4..5 of each lane
    };
    SmemT<kMNarrow / 4> narrow;
  };
  uint4 row[2][kNLet + 1];         // s and s+ of a bank-a letter, slots 0..19
  uint4 prev[2][kNLet + 1];        // s-, slots 20..29 (dwords 3, 4, 5), by half; entry kNLet: none
  union {
    uint8_t let[kSpan * kMRows];   // letters of the item's rows by step
    int16_t mat[kNLet * kNLet];    // while the tables are built
  };
  int32_t rowq[kMRows], rowseq[kMRows], rowpos[kMRows];
  uint32_t hit[kMWaves][kMSlots];  // row | score << 6 | column << 16
  int32_t n_hit[kMWaves];
  int32_t item;
  unsigned long long base;
};
static_assert(sizeof(MSmem) <= 80 * 1024, "two workgroups on a compute unit");

// E2M3 code of score / 2.
__device__ __forceinline__ uint32_t e2m3_half(int s) {
  const uint32_t v = (uint32_t)abs(s);
  // v / 2: 0.5 is subnormal (4 / 8), then mantissas of 3 bits with exponents 1, 2, 3
  const uint32_t c = v < 2 ? v * 4u : (v < 4 ? 8u + (v - 2) * 4u : (v < 8 ? 16u + (v - 4) * 2u : 24u + (v - 8)));
  return s < 0 ? c | 32u : c;
}

// Tables of the workgroup, once per launch (contains barriers and ends with one).
__device__ __forceinline__ void m_tables(const UngappedArgs& A, MSmem& S) {
  const int tid = threadIdx.x;
  for (int i = tid; i < kNLet * kNLet; i += kMThreads) S.mat[i] = A.mat[i];
  __syncthreads();
  for (int i = tid; i < 2 * (kNLet + 1); i += kMThreads) {
    const int h = i / (kNLet + 1), x = i % (kNLet + 1);
    unsigned long long lo = 0, hi = 0, v = 0;
#pragma unroll 1
    for (int c = 0; c < kPadCode; ++c) {
      const int s = x < kNLet ? S.mat[x * kNLet + c] : 0;
      const unsigned long long code = e2m3_half(h ? max(s, 0) : s);
      const int bit = 6 * c;
      if (bit < 64) lo |= code << bit;
      if (bit >= 64) hi |= code << (bit - 64);
      else if (bit > 58) hi |= code >> (64 - bit);
    }
#pragma unroll 1
    for (int c = 0; c < 10; ++c) {
      const int s = x < kNLet ? S.mat[x * kNLet + 10 * h + c] : 0;
      v |= (unsigned long long)e2m3_half(min(s, 0)) << (6 * c);
    }
    S.row[h][x] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    S.prev[h][x] = make_uint4((uint32_t)(v << 24), (uint32_t)(v >> 8), (uint32_t)(v >> 40), 0u);
  }
  for (int x = tid; x < kNLet; x += kMThreads) {
    uint32_t d[4] = {0, 0, 0, 0};
    if (x < kPadCode) d[x >> 3] = 4u << (4 * (x & 7));
    S.hot[0][x] = make_uint2(d[0], d[1]);
    S.hot[1][x] = make_uint2(d[2], d[3]);
    for (int h = 0; h < 2; ++h) {
      uint32_t e[4] = {0, 0, 0, 0};
      const int slot = 20 + x - 10 * h;
      if (x < kPadCode && slot >= 20 && slot < 30) e[slot >> 3] = 4u << (4 * (slot & 7));
      S.part[h][x] = make_uint2(e[2], e[3]);
    }
  }
  __syncthreads();
}

// Rows row0 .. row0 + rows - 1 of the key as profile operands of `tiles` tiles
// (rows past the item's are separators).  Contains barriers and ends with one.
__device__ __forceinline__ void m_profile(const UngappedArgs& A, const WorkItem& it, int64_t a0, int rows, int tiles,
                                          MSmem& S) {
  const int tid = threadIdx.x;
  if (tid < kMRows) {
    int q = -1, sq = 0, ps = 0;
    if (tid < rows) {
      const int64_t o = a0 + it.row0 + tid;
      q = A.a.occ[o];
      sq = A.a.occ_seq[o];
      ps = q - (int)A.a.seq_start[sq];
    }
    S.rowq[tid] = q;
    S.rowseq[tid] = sq;
    S.rowpos[tid] = ps;
  }
  __syncthreads();
  for (int i = tid; i < kSpan * kMRows; i += kMThreads) {
    const int t = i / kMRows, r = i % kMRows;
    const int q = S.rowq[r];
    int letter = kPadCode;
    if (q >= 0) letter = A.a.scan[t < kRight ? q + t : q - (t - kRight + 1)] / kScale;
    S.let[i] = (uint8_t)letter;
  }
  __syncthreads();
  const int lane = tid & 63, half = lane >> 5;
  for (int i = tid; i < tiles * kMSteps * 64; i += kMThreads) {
    const int k = (i >> 6) % kMSteps, t = (i >> 6) / kMSteps;
    const int r = t * kMTile + (lane & 31);
    const int x = S.let[(2 * k + half) * kMRows + r];
    const int y = k == 0 || k == kMRight ? kNLet : S.let[(2 * k - 1) * kMRows + r];
    const uint4 d = S.row[half][x], p = S.prev[half][y];
    S.a4[t][k][lane] = mu4{d.x, d.y, d.z, d.w | p.x};
    S.a2[t][k][lane] = mu2{p.y, p.z};
  }
  __syncthreads();
}

// One-hot operands of one side of the lane's column from its 44-letter window (as
// in scan_window: byte b is position q - 20 + b, letter * 8).
template <bool RIGHT, int N>
__device__ __forceinline__ void m_columns(const MSmem& S, const uint32_t (&win)[11], uint4 (&B)[N]) {
  const int half = __lane_id() >> 5;
  const uint8_t* hot = (const uint8_t*)S.hot;
  const uint8_t* part = (const uint8_t*)S.part[half];
  // shift of the letter of step 2k (lower half) or 2k + 1 (upper) in its dword, k even and odd
  const uint32_t s0 = RIGHT ? 8 * half : 24 - 8 * half, s1 = RIGHT ? 16 + 8 * half : 8 - 8 * half;
#pragma unroll
  for (int k = 0; k < (RIGHT ? kMRight : kMSteps - kMRight); ++k) {
    const int o = RIGHT ? kNbr + 2 * k : kNbr - 1 - 2 * k;  // byte of step 2k
    const int p = RIGHT ? o - 1 : o + 1;                    // byte of step 2k - 1
    const uint32_t x = __builtin_amdgcn_ubfe(win[o >> 2], k & 1 ? s1 : s0, 8);
    const uint2 d0 = *(const uint2*)(hot + x), d1 = *(const uint2*)(hot + x + sizeof(S.hot[0]));
    B[k] = make_uint4(d0.x, d0.y, d1.x, d1.y);
    if (k > 0) {
      const uint2 e = *(const uint2*)(part + ((win[p >> 2] >> (8 * (p & 3))) & 0xffu));
      B[k].z |= e.x;
      B[k].w = e.y;
    }
  }
}

// Read as volatile: two 8-byte reads are otherwise merged into one, whose four
// registers cannot be the tails of two operands, so that each MFMA pays a copy;
// and the operands of a tile are otherwise kept over the loop on the columns, in
// registers that there are not.
__device__ __forceinline__ mi8 m_profile_operand(const MSmem& S, int t, int k, int lane) {
  typedef const volatile __attribute__((address_space(3))) mu2* lds2;
  typedef const volatile __attribute__((address_space(3))) mu4* lds4;
  const mu4 x = *(lds4)&S.a4[t][k][lane];
  const mu2 y = *(lds2)&S.a2[t][k][lane];
  return mi8{(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)y.x, (int)y.y, 0, 0};
}

__device__ __forceinline__ mf16 m_step(const mi8& a, const uint4& b, const mf16& c) {
  const mi8 bb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, bb, c, 2, 4, 0, 0, 0, 0);
}

template <int FROM, int N>
__device__ __forceinline__ void m_max(mf16& m, const mf16& x, const mf16& y) {
#pragma unroll
  for (int i = FROM; i < FROM + N; ++i) m[i] = __builtin_fmaxf(__builtin_fmaxf(m[i], x[i]), y[i]);
}

// One side of tile t: the MFMAs FROM .. TO - 1 from the accumulators `start`,
// maxima into m (0 or `start` before).
template <int FROM, int TO, int N>
__device__ __forceinline__ void m_side(const MSmem& S, int t, int lane, const uint4 (&B)[N], const mf16& start,
                                       mf16& m) {
  mi8 a[TO - FROM];
#pragma unroll
  for (int k = 0; k < kMAhead; ++k) a[k] = m_profile_operand(S, t, FROM + k, lane);
  mf16 x0 = m_step(a[0], B[0], start);
  mf16 x1 = m_step(a[1], B[1], x0);
#pragma unroll
  for (int k = 2; k < TO - FROM; k += 2) {
#pragma unroll
    for (int j = k + kMAhead - 2; j < k + kMAhead; ++j)
      if (j < TO - FROM) a[j] = m_profile_operand(S, t, FROM + j, lane);
    const mf16 y0 = m_step(a[k], B[k], x1);
    __builtin_amdgcn_sched_barrier(0);
    m_max<0, 8>(m, x0, x1);
    __builtin_amdgcn_sched_barrier(0);
    const mf16 y1 = m_step(a[k + 1], B[k + 1], y0);
    __builtin_amdgcn_sched_barrier(0);
    m_max<8, 8>(m, x0, x1);
    __builtin_amdgcn_sched_barrier(0);
    x0 = y0;
    x1 = y1;
  }
  m_max<0, 16>(m, x0, x1);
  asm volatile("" : "+v"(m));  // the maxima stay here, and with them the accumulators' lifetimes
}

// Writes a wavefront's staged hits 0 .. n - 1 at hits[base ..).
__device__ __forceinline__ void m_write(const UngappedArgs& A, const MSmem& S, const WorkItem& it, int64_t b0, int wid,
                                        int n, unsigned long long base) {
  for (int e = __lane_id(); e < n; e += 64) {
    if (base + e >= (unsigned long long)A.capacity) continue;
    const uint32_t v = S.hit[wid][e];
    const int r = v & 63u;
    const int64_t o = b0 + it.col0 + (v >> 16);
    const int sq = A.b.occ_seq[o];
    plast_hit_t h;
    h.seq1 = S.rowseq[r];
    h.pos1 = S.rowpos[r];
    h.seq2 = sq;
    h.pos2 = A.b.occ[o] - (int)A.b.seq_start[sq];
    h.score = (int)((v >> 6) & 1023u);
    A.hits[base + e] = h;
  }
}

// Orders a wavefront's LDS accesses of its own staging area across lanes (the
// LDS serves one wavefront's instructions in order).
__device__ __forceinline__ void m_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Stages the hits of one accumulator register (row r in the lower half of the
// wavefront, r + 4 in the upper) from slot n on; returns how many.
__device__ __forceinline__ int m_stage(const UngappedArgs& A, MSmem& S, int wid, int r, int g, int n, unsigned long long hits, float score) {
  const int lane = __lane_id();
  if (score >= A.thrf) {
    const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
    S.hit[wid][at] = (uint32_t)(r + 4 * (lane >> 5)) | (uint32_t)(int)score << 6 |
                     (uint32_t)(g * 32 + (lane & 31)) << 16;
  }
  return __popcll(hits);
}

// The hits of a tile, counted.
__device__ __forceinline__ int m_count(const UngappedArgs& A, const mf16& m) {
  int total = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) total += (int)__popcll(__ballot(m[i] >= A.thrf));
  return total;
}

// The hits of tile t of the column group g, written at hits[at ..).
__device__ __forceinline__ void m_put(const UngappedArgs& A, const MSmem& S, const WorkItem& it, int64_t b0, int g, int t,
                                      unsigned long long at, const mf16& m) {
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));  // the addresses below are formed here, not kept in registers over the loop
  const int j = g * 32 + (lane & 31);
  const int64_t o = b0 + it.col0 + (j < it.ncols ? j : 0);  // (a column past the item's has no hit)
  plast_hit_t h;
  h.seq2 = A.b.occ_seq[o];
  h.pos2 = A.b.occ[o] - (int)A.b.seq_start[h.seq2];
  const int r0 = t * kMTile + 4 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const unsigned long long hits = __ballot(m[i] >= A.thrf);
    if (!hits) continue;
    const unsigned long long to =
        at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
    if (m[i] >= A.thrf && to < (unsigned long long)A.capacity) {
      h.seq1 = S.rowseq[r0 + 8 * (i / 4) + i % 4];
      h.pos1 = S.rowpos[r0 + 8 * (i / 4) + i % 4];
      h.score = (int)m[i];
      A.hits[to] = h;
    }
    at += __popcll(hits);
  }
}

// Finishes tile t of the column group g: its hits into the staging area (n staged
// before; returns how many are staged after).  `out` counts those written out; once they
// are many, `end`, which the groups go up to, becomes the next one.
// Register i holds rows 8 (i / 4) + i % 4 (lower half of the wavefront) and the ones 4
// below (upper half); one or two registers of a tile hold a hit, so four at a time are
// tested first.  A tile that may not fit the area is written out with the staged hits.
__device__ __forceinline__ int m_finish(const UngappedArgs& A, MSmem& S, const WorkItem& it, int64_t b0, int wid, int g,
                                        int t, int n, const mf16& m, int& out, int& end) {
  unsigned long long any[4];
  int most = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float top = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(m[4 * k], m[4 * k + 1]), m[4 * k + 2]), m[4 * k + 3]);
    any[k] = __ballot(top >= A.thrf);
    most += 4 * (int)__popcll(any[k]);
  }
  if (most == 0) return n;
  if (n + most > kMSlots) {
    const int total = m_count(A, m);
    if (n + total > kMSlots) {
      m_wave_sync();
      unsigned long long base = 0;
      if (__lane_id() == 0) base = atomicAdd(A.n_hits, (unsigned long long)(n + total));
      base = __shfl(base, 0);
      m_write(A, S, it, b0, wid, n, base);
      m_put(A, S, it, b0, g, t, base + n, m);
      m_wave_sync();
      out += n + total;
      if (out >= kMHotHits * ((g >> 2) + 1) && end - g > kMHotRest * kMWaves) end = g + 1;
      return 0;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!any[k]) continue;
#pragma unroll
    for (int i = 4 * k; i < 4 * k + 4; ++i) {
      const unsigned long long hits = __ballot(m[i] >= A.thrf);
      if (hits) n += m_stage(A, S, wid, t * kMTile + 8 * (i / 4) + i % 4, g, n, hits, m[i]);
    }
  }
  return n;
}

// An item of few rows on the VALU tile (contains barriers).
__device__ __forceinline__ void run_narrow(const UngappedArgs& A, const WorkItem& it, int64_t a0, int64_t b0, int rows,
                                           SmemT<kMNarrow / 4>& S) {
  smem_init<true, kMThreads>(A, S);  // its barrier comes with the profile
  if (rows <= 4)
    run_tile<true, 1, kMThreads>(A, it, a0, b0, rows, S);
  else
    run_tile<true, 2, kMThreads>(A, it, a0, b0, rows, S);
}

// All threads of the workgroup call run_item_m with the same item (it contains
// barriers).
//
// Hits are staged, and written out when the staging area is full or the item ends.
// Where they are many (banks that share low-complexity words, a low threshold), that is
// every few groups, and the atomics on the one counter, 14 ns each whoever makes them,
// take longer than the tiles: the rest of the wavefront's groups then runs twice, to
// count the hits and, with the room for them taken by one atomic, to write them.  1000 x
// 30,000 proteins at a threshold of 20 (117M hits): 1.76 ms, 11.4 without, 3.60 on the
// VALU tile; with runs over the same two letters in a tenth of both banks (1.12G hits)
// 5.0, 58.4 and 11.4 ms.
__device__ void run_item_m(const UngappedArgs& A, const WorkItem it, MSmem& S) {
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t a0 = A.a.key_off[it.key], b0 = A.b.key_off[it.key];
  const int n1 = (int)(A.a.key_off[it.key + 1] - a0);
  const int rows = __builtin_amdgcn_readfirstlane(min(kMRows, n1 - it.row0));
  if (rows <= kMNarrow) {
    run_narrow(A, it, a0, b0, rows, S.narrow);
    return;
  }
  const int tiles = (rows + kMTile - 1) / kMTile;
  m_profile(A, it, a0, rows, tiles, S);

  // Wavefront w takes the groups of 32 columns w, w + 4, ...; the occurrence two
  // groups ahead and the window one group ahead are in flight.
  const int groups = (it.ncols + 31) >> 5;
  const int c = lane & 31;
  auto occ_of = [&](int g) {
    const int j = g * 32 + c;
    return A.b.occ[b0 + it.col0 + (j < it.ncols ? j : 0)];
  };
  // The groups from `first` on, below `end`: finish(g, t, scores of tile t).
  auto scan = [&](int first, const int& end, auto finish) {
    int q = 0, q_nxt = 0;
    uint32_t raw[12];
    if (first < groups) {
      q = occ_of(first);
      load_window_raw(A, q, raw);
    }
    if (first + kMWaves < groups) q_nxt = occ_of(first + kMWaves);
    for (int g = first; g < end; g += kMWaves) {
      uint32_t win[11];
      const int sh = (q - kNbr) & 3;
#pragma unroll
      for (int i = 0; i < 11; ++i) win[i] = __builtin_amdgcn_alignbyte(raw[i + 1], raw[i], sh);
      // A column past the item's is a window of separators: it scores 0, like a
      // row past the item's, and 0 is below the threshold.
      if (it.ncols - g * 32 < 32) {
#pragma unroll
        for (int i = 0; i < 11; ++i) win[i] = g * 32 + c < it.ncols ? win[i] : kPadCode * kScale * 0x01010101u;
      }
      uint4 B[kMRight];
      mf16 m0, m1;
#pragma unroll
      for (int i = 0; i < 16; ++i) m0[i] = m1[i] = 0.f;
      m_columns<true>(S, win, B);
      if (g + kMWaves < groups) {
        q = q_nxt;
        load_window_raw(A, q, raw);
      }
      if (g + 2 * kMWaves < groups) q_nxt = occ_of(g + 2 * kMWaves);
      const mf16 zero = m0;
      m_side<0, kMRight>(S, 0, lane, B, zero, m0);
      if (tiles > 1) m_side<0, kMRight>(S, 1, lane, B, zero, m1);
      m_columns<false>(S, win, B);
      const mf16 r0 = m0, r1 = m1;
      m_side<kMRight, kMSteps>(S, 0, lane, B, r0, m0);
      finish(g, 0, m0);
      if (tiles > 1) {
        m_side<kMRight, kMSteps>(S, 1, lane, B, r1, m1);
        finish(g, 1, m1);
      }
    }
  };
  int n = 0, out = 0;              // hits staged now, and written out before
  int end = groups;
  scan(wid, end, [&](int g, int t, const mf16& m) { n = m_finish(A, S, it, b0, wid, g, t, n, m, out, end); });
  if (end < groups) {
    const int rest = end - 1 + kMWaves;
    int counted = 0;
    unsigned long long at = 0;     // where they go
    bool write = false;
    for (;;) {
      scan(rest, groups,
           [&](int g, int t, const mf16& m) {
             const int hits = m_count(A, m);
             if (!write) {
               counted += hits;
             } else if (hits) {
               m_put(A, S, it, b0, g, t, at, m);
               at += hits;
             }
           });
      if (write || counted == 0) break;
      if (lane == 0) at = atomicAdd(A.n_hits, (unsigned long long)counted);
      at = __shfl(at, 0);
      write = true;
    }
  }
  // the item's hits go out with one global atomic
  if (lane == 0) S.n_hit[wid] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    int total = 0;
    for (int w = 0; w < kMWaves; ++w) total += S.n_hit[w];
    S.base = total ? atomicAdd(A.n_hits, (unsigned long long)total) : 0ull;
  }
  __syncthreads();
  unsigned long long base = S.base;
  for (int w = 0; w < wid; ++w) base += S.n_hit[w];
  m_write(A, S, it, b0, wid, n, base);
  __syncthreads();
}
