// The ungapped extension with a work item per wavefront (included by
// ungapped.hip, inside its namespace), for small banks.
//
// With a few hundred proteins on both sides a key has a handful of rows and tens
// of columns: a workgroup of 512 on such an item idles on all but a few lanes,
// spends about 9 us on the item's chain of loads and barriers, and the atomic that
// hands out items, about 12 ns each on one address, takes as long as the pairs.
// Here every wavefront takes items of its own, by striding over the list: 16
// wavefronts on a compute unit, each with the profile of 4 rows at a time (7 KB of
// LDS) and a staging area for its hits, and no barrier before the end, when the hits
// that are left in a workgroup are written with one global atomic.  Bound by the
// latency of the loads that an item begins with (work list, key table, occurrences,
// letters).
//
// A list of fewer items than wavefronts is cut further, into slices of the items'
// columns.  Where bank b is larger than an L2, a column's window comes from a random
// place past it; while an eighth of the bank about fits one, each XCD takes the columns
// of its eighth of the bank.
//
// Measured, against a workgroup per item (proteins, us): 200 x 2000 63 and 162, 30 x
// 2000 28 and 72, 3 x 300 14 and 22, 100 x 10,000 103 and 175, 3 x 100,000 88 and 130
// (112 without the XCDs' shares), 30 x 100,000 290 and 466 (418), 3 x 1M 1116 and 1533.
constexpr int kWWaves = kThreads / 64;
static_assert(kXcds == kMaxQueues, "an eighth of the columns, and a queue, an XCD");
// Keys whose items are large (many rows of many columns) are left to the workgroups, as
// in the kernel of an item per workgroup, once their wavefronts have ended: the 32-row
// tile reads a window once for 32 rows instead of 4, and shares an item of many hits
// between 8 wavefronts.  Banks whose sequences share low-complexity words have a few such
// keys whatever their size.  Rows x columns of an item from which that pays, where a
// wavefront takes up to half of an item's columns (200 x 10,000 proteins 148 us, from
// 8192 on 141, from 32768 164, and 189 with none; 30 x 100,000 285, 351, 299 and 350; 10 x
// 300,000 742, 766, 765 and 755), more where it takes fewer, and three times as many
// where there are few pairs in all, as the product of the words says, since what is left
// to the end then takes as long as all else (100 proteins x 60,000 fragments 50 and 56
// us).  With runs over the same two letters in a tenth of 200 x 10,000 proteins 0.97 ms,
// 4.5 with no such keys.
constexpr int kWLarge = 16384;
constexpr double kWFew = 3e10;
constexpr int kWLargeCols = 4096;  // columns of an item that count: the wider ones of 1 to 3 rows stay
constexpr int kWMatRow = 22;                        // entries of a matrix row in LDS: dwords of two letters
constexpr int kWRows = 8;                           // rows of an item that a wavefront takes at a time
constexpr int kWSlices = 16;                        // most slices of an item's columns

// Hits are staged by each wavefront as occurrence indexes and a score: as many as a
// group of 64 columns and 4 rows can have, so that a group always fits an empty area.
// (One area of 512 a workgroup, written out at the end alone, left every group that found
// it full an atomic of its own, 14 ns each on the one counter: 200 x 10,000 proteins at a
// threshold of 25 instead of 38 took 1.92 ms, 0.24 now.)
constexpr int kWSlots = 4 * 64;

// Slices of an item's columns in a list of n_items.  A wavefront of the launch takes 1 of
// `waves` items, or those of its XCD's eighth of the columns.
__host__ __device__ inline int w_slices(bool xcd, int64_t waves, int64_t n_items) {
  return (int)min((int64_t)kWSlices, 1 + (xcd ? 8 : 4) * waves / max(n_items, (int64_t)1));
}

// PlanShape::large, for as many items as banks of ordinary sequences make.
inline int w_large(const plast_index_t* a, const plast_index_t* b, const plast_tuning_t& t, int grid) {
  const int64_t n2 = (int64_t)(words_of(b) / kNKeys);
  int c = 0;
  for (int i = 1; i < kClasses; ++i)
    if (n2 >= t.class_min_n2[i]) c = i;
  const int64_t n_items = min((int64_t)words_of(a), (int64_t)kNKeys) * (n2 / t.item_cols[c] + 1);
  const bool xcd = columns_shared(b->n_padded, grid);
  const int slices = w_slices(xcd, (int64_t)grid * kWWaves / (xcd ? kMaxQueues : 1), n_items);
  return kWLarge * max(slices / 2, 1) * (words_of(a) * words_of(b) < kWFew ? 3 : 1);
}

struct __align__(16) WSmem {
  uint8_t prof[kWWaves][kProfRG];      // 8-byte entries
  uint16_t mat[kNLet * kWMatRow];      // profile values (int16 or binary16 bits)
  int32_t hit_a[kWWaves][kWSlots], hit_b[kWWaves][kWSlots];
  uint16_t hit_score[kWWaves][kWSlots];
  int32_t n_hit[kWWaves];              // staged when the wavefront has ended
  unsigned long long base;
};
static_assert(sizeof(WSmem) <= 80 * 1024, "two workgroups on a compute unit");
static_assert(kSpan * 128 < 1 << 16, "a staged score has 16 bits");

__device__ __forceinline__ void w_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Writes a wavefront's staged hits 0 .. n - 1 at hits[base ..).
__device__ __forceinline__ void w_write(const UngappedArgs& A, const WSmem& S, int wid, int n,
                                        unsigned long long base) {
  for (int e = __lane_id(); e < n; e += 64) {
    if (base + e >= (unsigned long long)A.capacity) continue;
    const int oa = S.hit_a[wid][e], ob = S.hit_b[wid][e];
    plast_hit_t h;
    h.seq1 = A.a.occ_seq[oa];
    h.pos1 = A.a.occ[oa] - (int)A.a.seq_start[h.seq1];
    h.seq2 = A.b.occ_seq[ob];
    h.pos2 = A.b.occ[ob] - (int)A.b.seq_start[h.seq2];
    h.score = S.hit_score[wid][e];
    A.hits[base + e] = h;
  }
}

// Stages the hits of one column per lane against 4 rows (row r of register r / 2)
// after the n staged before, which are written out first, with one global atomic, if
// the new ones do not fit beside them.  Returns how many are staged then.  All lanes
// call it.
template <bool F16>
__device__ __forceinline__ int w_hits(const UngappedArgs& A, WSmem& S, const vec2<F16> (&m)[2], uint32_t mask, int oa,
                                      int ob, int wid, int n) {
  unsigned long long b[4];
  int total = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    b[r] = __ballot((mask & row_bit(r)) != 0);
    total += (int)__popcll(b[r]);
  }
  if (total == 0) return n;
  if (n + total > kWSlots) {
    w_sync();
    unsigned long long base = 0;
    if (__lane_id() == 0) base = atomicAdd(A.n_hits, (unsigned long long)n);
    w_write(A, S, wid, n, __shfl(base, 0));
    w_sync();
    n = 0;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (mask & row_bit(r)) {
      const int at =
          n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[r], 0u));
      S.hit_a[wid][at] = oa + r;
      S.hit_b[wid][at] = ob;
      S.hit_score[wid][at] = (uint16_t)to_int<F16>(m[r / 2], r & 1);
    }
    n += (int)__popcll(b[r]);
  }
  return n;
}

// Rows row .. row + kWRows - 1 of an item (those that it has; ka and ka1: its key's
// first occurrence in bank a and the next key's, kb: its first in bank b) against
// the columns from .. to - 1 of the key in groups of 64, every slices-th of them.
// n hits are staged before; returns how many are after.
template <bool F16>
__device__ __forceinline__ int run_item_w(const UngappedArgs& A, const WorkItem it, int64_t ka, int64_t ka1, int64_t kb,
                                          int row, int from, int to, int slices, int wid, int n, WSmem& S) {
  const int lane = __lane_id();
  const int a0 = (int)ka + it.row0 + row, b0 = (int)kb;
  const int rows = min(min(kWRows, kTileRows - row), (int)ka1 - a0);
  if (rows <= 0 || from >= to) return n;
  const int qrow = lane < rows ? A.a.occ[a0 + lane] : -1;
  uint8_t* prof = S.prof[wid];
  for (int r0 = 0; r0 < rows; r0 += 4) {
    w_sync();  // the profile before is read
    // Lane t writes the entries of scan step t: the scores of the 4 rows against two
    // letters at a time, from the rows' letters at that step.
    if (lane < kSpan) {
      const int off = lane < kRight ? lane : -(lane - kRight + 1);
      const uint32_t* row_of[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = __builtin_amdgcn_readlane(qrow, r0 + r);
        const uint32_t letter = q >= 0 ? A.a.scan[q + off] / kScale : (uint32_t)kPadCode;
        row_of[r] = (const uint32_t*)S.mat + letter * (kWMatRow / 2);
      }
      uint8_t* dst = prof + lane * kProfT;
#pragma unroll
      for (int c = 0; c < kNLet; c += 2) {
        const uint32_t w0 = row_of[0][c / 2], w1 = row_of[1][c / 2], w2 = row_of[2][c / 2], w3 = row_of[3][c / 2];
        *(uint2*)(dst + c * 8) = make_uint2(__builtin_amdgcn_perm(w1, w0, 0x05040100u), __builtin_amdgcn_perm(w3, w2, 0x05040100u));
        if (c + 1 < kNLet)
          *(uint2*)(dst + (c + 1) * 8) = make_uint2(__builtin_amdgcn_perm(w1, w0, 0x07060302u), __builtin_amdgcn_perm(w3, w2, 0x07060302u));
      }
    }
    w_sync();
    const uint32_t valid = valid_rows_mask(min(4, rows - r0));
    // the next group's occurrence and window are in flight
    auto occ_of = [&](int c0) { return b0 + min(c0 + lane, to - 1); };
    int q2 = A.b.occ[occ_of(from)];
    uint32_t raw[12];
    load_window_raw(A, q2, raw);
    for (int c0 = from; c0 < to; c0 += slices * 64) {
      const bool active = c0 + lane < to;
      const int ob = occ_of(c0);
      uint32_t win[11];
      const int sh = (q2 - kNbr) & 3;
#pragma unroll
      for (int i = 0; i < 11; ++i) win[i] = __builtin_amdgcn_alignbyte(raw[i + 1], raw[i], sh);
      if (c0 + slices * 64 < to) {
        q2 = A.b.occ[occ_of(c0 + slices * 64)];
        load_window_raw(A, q2, raw);
      }
      vec2<F16> m[2];
      scan_window<F16, 1>(prof, win, m);
      n = w_hits<F16>(A, S, m, active ? (hit_mask<F16, 1>(A.thr, m) & valid) : 0u, a0 + r0, ob, wid, n);
    }
  }
  return n;
}

template <bool F16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_ungapped_wave(UngappedArgs A, const WorkItem* __restrict__ items, const UngappedCounters* __restrict__ cnt,
                     const int32_t* __restrict__ list_len, int32_t* __restrict__ ctr, int32_t n_queues, bool xcd) {
  __shared__ union {
    WSmem wave;
    Smem group;
  } L;
  WSmem& S = L.wave;
  for (int i = threadIdx.x; i < kNLet * kNLet; i += kThreads) {
    uint16_t v;
    if constexpr (F16)
      v = __builtin_bit_cast(uint16_t, (_Float16)A.mat[i]);
    else
      v = (uint16_t)A.mat[i];
    S.mat[i / kNLet * kWMatRow + i % kNLet] = v;
  }
  __syncthreads();
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_large = __builtin_amdgcn_readfirstlane(cnt->overflow ? 0 : list_len[1]);
  const int n_items = __builtin_amdgcn_readfirstlane(cnt->overflow ? 0 : list_len[0]) - n_large;
  const WorkItem* __restrict__ large = items;
  items += n_large;
  int n = 0;  // staged hits
  if (xcd) {
    // Each XCD (workgroups are dealt to them round robin) takes an eighth of every
    // key's columns, which lie in the same eighth of the bank: its L2 then serves
    // most windows.  A unit is a slice of an item's columns there.
    const int x = blockIdx.x % kMaxQueues;
    const int waves = ((int)gridDim.x - x + kMaxQueues - 1) / kMaxQueues * kWWaves;
    const int slices = w_slices(true, waves, n_items);
    const int64_t n_units = (int64_t)n_items * slices;
    for (int64_t u = (int64_t)(blockIdx.x / kMaxQueues) * kWWaves + wid; u < n_units; u += waves) {
      const WorkItem it = items[u % n_items];
      const int64_t ka = A.a.key_off[it.key], ka1 = A.a.key_off[it.key + 1];
      const int64_t kb = A.b.key_off[it.key], n2 = A.b.key_off[it.key + 1] - kb;
      const int from = max(it.col0, (int)(n2 * x / kMaxQueues));
      const int to = min(it.col0 + it.ncols, (int)(n2 * (x + 1) / kMaxQueues));
      for (int row = 0; row < kTileRows; row += kWRows)
        n = run_item_w<F16>(A, it, ka, ka1, kb, row, from + (int)(u / n_items) * 64, to, slices, wid, n, S);
    }
  } else {
    // units of kWRows rows of an item, most of which have fewer rows in all
    constexpr int kUnits = kTileRows / kWRows;
    const int64_t stride = (int64_t)gridDim.x * kWWaves;
    // and of a slice of its columns where the list has few items for the wavefronts
    const int slices = w_slices(false, stride, n_items);
    const int64_t n_units = (int64_t)n_items * kUnits * slices;
    for (int64_t u = (int64_t)blockIdx.x * kWWaves + wid; u < n_units; u += stride) {
      // all first units before all second ones: neighbouring wavefronts have like work
      const int i = (int)(u % n_items), part = (int)(u / n_items);
      const WorkItem it = items[i];
      n = run_item_w<F16>(A, it, A.a.key_off[it.key], A.a.key_off[it.key + 1], A.b.key_off[it.key],
                          part / slices * kWRows, it.col0 + part % slices * 64, it.col0 + it.ncols, slices, wid, n, S);
    }
  }
  // what the wavefronts have left goes out with one global atomic
  if (__lane_id() == 0) S.n_hit[wid] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    int total = 0;
    for (int w = 0; w < kWWaves; ++w) total += S.n_hit[w];
    S.base = total ? atomicAdd(A.n_hits, (unsigned long long)total) : 0ull;
  }
  __syncthreads();
  unsigned long long base = S.base;
  for (int w = 0; w < wid; ++w) base += S.n_hit[w];
  w_write(A, S, wid, n, base);
  if (n_large == 0) return;
  __syncthreads();
  smem_init<F16, kThreads>(A, L.group);  // its barrier comes with the first item
  work_loop(n_large, ctr, n_queues, &L.group.item, [&](int i) { run_item<F16>(A, large[i], L.group); });
}
