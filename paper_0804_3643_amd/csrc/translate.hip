// TPLAST-N (Sec. 6): six-frame translation of a nucleotide bank on the device.
//
// Frames 0..2 read the forward strand from nucleotide 0, 1 or 2; frames 3..5
// read the reverse complement the same way; a trailing partial codon is
// dropped.  The standard genetic code maps each codon to an amino acid or a
// stop, and stops cut every frame into fragments; each non-empty fragment
// becomes one protein sequence of the output bank (padded layout), so that seed
// windows never cross a stop.  Fragment j is described by (DNA sequence, frame,
// offset of its first amino acid in the frame).
//
// One workgroup per (sequence, frame) stream.  Pass 1 counts the stream's
// fragments and amino acids; an exclusive scan over the streams gives each
// stream its first fragment and first residue; pass 2 writes every amino acid
// to 20 (fragment + 1) + (residues before it), since the layout is a separator
// run, fragment 0, a run, fragment 1, ... .
//
// In both passes a thread takes 16 consecutive codons: 48 nucleotides in three
// 16-byte loads, a codon's index from one or two v_dot4 of its bytes with the
// weights of its bases, and its amino acid from a 64-byte table in LDS.  In pass
// 2 a workgroup scans its threads' counts, builds the bytes of its chunk (the
// separator runs included) in LDS and copies them out as dwords, so every byte
// of the bank is written once.  Bound by the loads and stores: 300 sequences of
// 50-200 kb (37 Mnt, 158 MB written) take 0.065 + 0.195 ms, where loads by the byte,
// a table in the kernel's arguments and byte stores over a separator fill took
// 0.46 + 0.34.
#include <stddef.h>

#include "plast_internal.h"

namespace plast {

namespace {

// Standard genetic code (NCBI table 1): the amino acid of codon b1 b2 b3, bases
// in the order A C G T, first base slowest; '*' = stop.  This library's
// transcription.
constexpr char kCodeACGT[65] = "KNKNTTTTRSRSIIMIQHQHPPPPRRRRLLLLEDEDAAAAGGGGVVVV*Y*YSSSS*CWCLFLF";
constexpr uint8_t kStop = 0xff;
// Workgroups of 256 threads, 4096 codons at a time; of 64 threads where the
// sequences are short on average (reads, ESTs, genes), since a stream of 250 codons
// fills 16 threads: 3000 sequences of 4-16 kb take 0.21 ms with 64, 0.29 with 256;
// 300 of 50-200 kb, whose 1800 streams are too few for one wavefront each, 0.49 and
// 0.29.
constexpr int kTrLong = 256, kTrShort = 64;
constexpr int kTrPer = 16;                         // codons of a thread
constexpr int64_t kTrShortNt = 16384;              // mean nucleotides up to which 64 threads are taken

struct CodonTable {
  uint8_t aa[64];  // residue code (ACDEFGHIKLMNPQRSTVWY order) or kStop
};

CodonTable codon_table() {
  static const char* kOrder = "ACDEFGHIKLMNPQRSTVWY";
  CodonTable t;
  for (int i = 0; i < 64; ++i) {
    const char c = kCodeACGT[i];
    t.aa[i] = kStop;
    for (int k = 0; k < 20; ++k)
      if (kOrder[k] == c) t.aa[i] = (uint8_t)k;
  }
  return t;
}

struct Stream {
  int64_t start, len;  // the DNA sequence
  int frame;
  int64_t n_codons;
};

__device__ __forceinline__ Stream stream_of(const int64_t* __restrict__ dna_start, int32_t n_dna, int64_t n_nt,
                                            int s, int32_t* __restrict__ err) {
  Stream S;
  const int d = s / 6;
  S.frame = s % 6;
  S.start = dna_start[d];
  const int64_t end = dna_start[d + 1];
  S.len = end - S.start;
  if (S.start < 0 || end > n_nt || S.len < 0) {  // inconsistent offsets: an empty stream
    if (threadIdx.x == 0 && S.frame == 0) atomicOr(err, 1);
    S.start = 0;
    S.len = 0;
  }
  const int off = S.frame % 3;
  S.n_codons = S.len > off ? (S.len - off) / 3 : 0;
  return S;
}

// The codon table in LDS (called by all threads; a barrier must follow).
__device__ __forceinline__ void table_to_lds(const CodonTable& T, uint8_t* aa) {
  if (threadIdx.x < 64) aa[threadIdx.x] = T.aa[threadIdx.x];
}

// Residue codes (kStop for stops and past the stream's end) of codons i0 ..
// i0 + 15 of a stream, four to a dword.
__device__ __forceinline__ void load_codons(const uint8_t* __restrict__ dna, int64_t n_nt, const Stream& S, int64_t i0,
                                            const uint8_t* aa, uint32_t (&out)[kTrPer / 4]) {
  const int64_t left = S.n_codons - i0;
  if (left <= 0) {
#pragma unroll
    for (int g = 0; g < kTrPer / 4; ++g) out[g] = ~0u;
    return;
  }
  const bool fwd = S.frame < 3;
  // first forward position of the 48 nucleotides: the frame's strand position
  // 3 i0 (+ offset) or, on the reverse strand, 47 before its forward position
  const int64_t q = S.frame % 3 + 3 * i0;
  const int64_t p = S.start + (fwd ? q : S.len - 48 - q);
  uint32_t w[12];
  if (p >= 0 && p + 48 <= n_nt) {
    __builtin_memcpy(w, dna + p, 48);
  } else {  // the bank's ends
#pragma unroll
    for (int d = 0; d < 12; ++d) {
      w[d] = 0;
      for (int k = 0; k < 4; ++k) {
        const int64_t x = p + 4 * d + k;
        if (x >= 0 && x < n_nt) w[d] |= (uint32_t)dna[x] << (8 * k);
      }
    }
  }
  // weights of a codon's bytes in memory order (first byte lowest)
  const uint32_t c0 = fwd ? 16u : 1u, c1 = 4u, c2 = fwd ? 1u : 16u;
  const uint32_t flip = fwd ? 0u : 63u;  // the reverse strand reads complements
#pragma unroll
  for (int g = 0; g < kTrPer / 4; ++g) {
    const uint32_t a = w[3 * g], b = w[3 * g + 1], c = w[3 * g + 2];
    uint32_t idx[4];
    idx[0] = __builtin_amdgcn_udot4(a, c0 | c1 << 8 | c2 << 16, 0u, false);
    idx[1] = __builtin_amdgcn_udot4(b, c1 | c2 << 8, __builtin_amdgcn_udot4(a, c0 << 24, 0u, false), false);
    idx[2] = __builtin_amdgcn_udot4(c, c2, __builtin_amdgcn_udot4(b, c0 << 16 | c1 << 24, 0u, false), false);
    idx[3] = __builtin_amdgcn_udot4(c, c0 << 8 | c1 << 16 | c2 << 24, 0u, false);
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = aa[(idx[k] ^ flip) & 63u];
    // the reverse strand's codon order is memory's reversed
    out[fwd ? g : kTrPer / 4 - 1 - g] =
        fwd ? (r[0] | r[1] << 8 | r[2] << 16 | r[3] << 24) : (r[3] | r[2] << 8 | r[1] << 16 | r[0] << 24);
  }
  if (left < kTrPer) {
#pragma unroll
    for (int k = 0; k < kTrPer; ++k)
      if (k >= left) out[k / 4] |= 0xffu << (8 * (k % 4));
  }
}

// Bit k of the result: codon k of the 16 is an amino acid.
__device__ __forceinline__ uint32_t live_mask(const uint32_t (&aa)[kTrPer / 4]) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < kTrPer; ++k) m |= (((aa[k / 4] >> (8 * (k % 4) + 7)) & 1u) ^ 1u) << k;
  return m;
}

// Whether codon i0 - 1 of the stream is an amino acid (i0 > 0), from the thread
// before this one, or read by a wavefront's first thread.
__device__ __forceinline__ bool live_before(const uint8_t* __restrict__ dna, const Stream& S, int64_t i0, uint32_t live,
                                            const uint8_t* aa) {
  const uint32_t up = __shfl_up(live, 1);
  if (__lane_id() != 0) return (up >> (kTrPer - 1)) & 1u;
  if (i0 == 0 || i0 > S.n_codons) return false;
  const int64_t q = S.frame % 3 + 3 * (i0 - 1);
  uint32_t b1, b2, b3;
  if (S.frame < 3) {
    const uint8_t* p = dna + S.start + q;
    b1 = p[0];
    b2 = p[1];
    b3 = p[2];
  } else {
    const uint8_t* p = dna + S.start + S.len - 1 - q;
    b1 = 3u - p[0];
    b2 = 3u - p[-1];
    b3 = 3u - p[-2];
  }
  return aa[((b1 & 3u) << 4) | ((b2 & 3u) << 2) | (b3 & 3u)] != kStop;
}

// Workgroup-wide inclusive scan of v (all threads call it; contains barriers).
template <int NT>
__device__ __forceinline__ int block_incl_sum(int v, int* wtot, int* total) {
  const int w = threadIdx.x >> 6, lane = __lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o);
    if (lane >= o) v += t;
  }
  if (lane == 63) wtot[w] = v;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    before += k < w ? wtot[k] : 0;
    all += wtot[k];
  }
  __syncthreads();
  *total = all;
  return before + v;
}

// Workgroup-wide sum (all threads call it; contains barriers).
template <int NT>
__device__ __forceinline__ long long block_sum64(long long v, long long* wsum) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
  __syncthreads();  // wsum may still be read by a previous call
  if (__lane_id() == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  long long t = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) t += wsum[k];
  return t;
}

// Pass 1: per stream, fragments and amino acids; frame-0 workgroups also check
// that every nucleotide code is 0..3.
template <int NT>
__global__ __launch_bounds__(NT) void k_tr_count(const uint8_t* __restrict__ dna,
                                                 const int64_t* __restrict__ dna_start, int32_t n_dna, int64_t n_nt,
                                                 CodonTable T, int64_t* __restrict__ nfrag,
                                                 int64_t* __restrict__ nres, int32_t* __restrict__ err) {
  __shared__ long long wsum[NT / 64];
  __shared__ uint8_t aa[64];
  table_to_lds(T, aa);
  __syncthreads();
  const int s = blockIdx.x;
  const Stream S = stream_of(dna_start, n_dna, n_nt, s, err);
  if (S.frame == 0) {
    uint32_t bad = 0;
    int64_t p = 16 * (int64_t)threadIdx.x;
    for (; p + 16 <= S.len; p += 16 * NT) {
      uint32_t w[4];
      __builtin_memcpy(w, dna + S.start + p, 16);
      bad |= (w[0] | w[1] | w[2] | w[3]) & 0xfcfcfcfcu;
    }
    for (; p < S.len; ++p) bad |= dna[S.start + p] > 3;  // the last, partial 16 of one thread
    if (bad) atomicOr(err, 2);
  }
  // each thread counts its own codons; one sum over the workgroup at the end
  long long frags = 0, res = 0;
  for (int64_t base = 0; base < S.n_codons; base += kTrPer * NT) {
    const int64_t i0 = base + kTrPer * (int64_t)threadIdx.x;
    uint32_t c[kTrPer / 4];
    load_codons(dna, n_nt, S, i0, aa, c);
    const uint32_t live = live_mask(c);
    const uint32_t first = live & ~(live << 1 | (uint32_t)live_before(dna, S, i0, live, aa));
    frags += __popc(first);
    res += __popc(live);
  }
  frags = block_sum64<NT>(frags, wsum);
  res = block_sum64<NT>(res, wsum);
  if (threadIdx.x == 0) {
    nfrag[s] = frags;
    nres[s] = res;
  }
}

// Exclusive scans of both counts over the streams, totals at [n] and beside the
// error word (one copy to the host).  Up to kScanParts workgroups take equal
// parts; with more than one, k_tr_part has summed the parts before.  (One
// workgroup took most of 2.35 ms for 40,000 reads, 0.56 now.)
constexpr int kTrScanThreads = 1024;
constexpr int kScanParts = 15;

struct TrHeader {
  int32_t err, pad;
  int64_t frags, res;               // totals
  int64_t part[kScanParts - 1][2];  // sums of the parts (the last one's is not needed)
};
static_assert(sizeof(TrHeader) <= 256, "translation header");

__host__ __device__ __forceinline__ int scan_part_begin(int n, int parts, int k) { return (int)((int64_t)n * k / parts); }

__global__ __launch_bounds__(kTrScanThreads) void k_tr_part(const int64_t* __restrict__ nfrag,
                                                            const int64_t* __restrict__ nres, int n, int parts,
                                                            TrHeader* __restrict__ H) {
  __shared__ long long wsum[kTrScanThreads / 64];
  long long f = 0, r = 0;
  for (int i = scan_part_begin(n, parts, blockIdx.x) + threadIdx.x; i < scan_part_begin(n, parts, blockIdx.x + 1);
       i += kTrScanThreads) {
    f += nfrag[i];
    r += nres[i];
  }
  f = block_sum64<kTrScanThreads>(f, wsum);
  r = block_sum64<kTrScanThreads>(r, wsum);
  if (threadIdx.x == 0 && blockIdx.x < kScanParts - 1) {
    H->part[blockIdx.x][0] = f;
    H->part[blockIdx.x][1] = r;
  }
}

__global__ __launch_bounds__(kTrScanThreads) void k_tr_scan(int64_t* __restrict__ nfrag, int64_t* __restrict__ nres,
                                                            int n, int parts, TrHeader* __restrict__ H) {
  __shared__ long long wsum[2][kTrScanThreads / 64];
  const int w = threadIdx.x >> 6, lane = __lane_id();
  long long carry[2] = {0, 0};
  for (int k = 0; k < (int)blockIdx.x; ++k) {
    carry[0] += H->part[k][0];
    carry[1] += H->part[k][1];
  }
  const int end = scan_part_begin(n, parts, blockIdx.x + 1);
  for (int base = scan_part_begin(n, parts, blockIdx.x); base < end; base += kTrScanThreads) {
    const int s = base + threadIdx.x;
    const long long own[2] = {s < end ? nfrag[s] : 0, s < end ? nres[s] : 0};
    long long v[2] = {own[0], own[1]};
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long a = __shfl_up(v[0], o), b = __shfl_up(v[1], o);
      if (lane >= o) {
        v[0] += a;
        v[1] += b;
      }
    }
    if (lane == 63) {
      wsum[0][w] = v[0];
      wsum[1][w] = v[1];
    }
    __syncthreads();
    long long all[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < kTrScanThreads / 64; ++k) {
      for (int x = 0; x < 2; ++x) {
        v[x] += k < w ? wsum[x][k] : 0;
        all[x] += wsum[x][k];
      }
    }
    if (s < end) {
      nfrag[s] = carry[0] + v[0] - own[0];
      nres[s] = carry[1] + v[1] - own[1];
    }
    carry[0] += all[0];
    carry[1] += all[1];
    __syncthreads();
  }
  if (threadIdx.x == 0 && (int)blockIdx.x == parts - 1) {
    nfrag[n] = H->frags = carry[0];
    nres[n] = H->res = carry[1];
  }
}

__global__ void k_tr_clear(int32_t* __restrict__ err) {
  if (threadIdx.x == 0) *err = 0;
}

// The bank of no sequences.
__global__ void k_tr_pad(uint8_t* __restrict__ codes, int64_t n, int64_t* __restrict__ seq_start, int64_t n_frags) {
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) codes[i] = kPadCode;
  if (threadIdx.x == 0) seq_start[n_frags] = n;
}

// Pass 2: the bank's bytes, fragment starts and the fragment table.
template <int NT>
__global__ __launch_bounds__(NT) void k_tr_write(const uint8_t* __restrict__ dna,
                                                 const int64_t* __restrict__ dna_start, int32_t n_dna, int64_t n_nt,
                                                 CodonTable T, const int64_t* __restrict__ frag0,
                                                 const int64_t* __restrict__ res0, uint8_t* __restrict__ codes,
                                                 int64_t n_padded, int64_t* __restrict__ seq_start,
                                                 int32_t* __restrict__ frag, int64_t n_frags,
                                                 int32_t* __restrict__ err) {
  // A chunk of n codons with r amino acids in f fragments writes 20 f + r bytes,
  // f <= r <= n - f + 1: at most 21 (n + 1) / 2.
  constexpr int kCodons = NT * kTrPer;
  constexpr int kMaxBytes = (1 + kPadLen) * (kCodons / 2 + 1);
  __shared__ __align__(16) uint8_t buf[(kMaxBytes + 4 + 15) / 16 * 16];
  __shared__ int wtot[NT / 64];
  __shared__ uint8_t aa[64];
  table_to_lds(T, aa);
  const int s = blockIdx.x;
  // what follows the last fragment
  const int64_t used = (int64_t)kPadLen * frag0[6 * (int64_t)n_dna] + res0[6 * (int64_t)n_dna];
  for (int64_t i = used + (int64_t)blockIdx.x * NT + threadIdx.x; i < n_padded; i += (int64_t)gridDim.x * NT)
    codes[i] = kPadCode;
  if (s == 0 && threadIdx.x == 0) seq_start[n_frags] = n_padded;
  const Stream S = stream_of(dna_start, n_dna, n_nt, s, err);
  int64_t cf = frag0[s], cr = res0[s];  // fragments and residues before this chunk
  __syncthreads();
  for (int64_t base = 0; base < S.n_codons; base += kCodons) {
    const int64_t i0 = base + kTrPer * (int64_t)threadIdx.x;
    uint32_t c[kTrPer / 4];
    load_codons(dna, n_nt, S, i0, aa, c);
    const uint32_t live = live_mask(c);
    const uint32_t first = live & ~(live << 1 | (uint32_t)live_before(dna, S, i0, live, aa));
    const int mine = (__popc(first) << 16) | __popc(live);
    int tot = 0;
    const int excl = block_incl_sum<NT>(mine, wtot, &tot) - mine;
    // the chunk's bytes [g0, g0 + bytes) of the bank, staged at their place modulo 4
    const int64_t g0 = (int64_t)kPadLen * cf + cr;
    const int bytes = kPadLen * (tot >> 16) + (tot & 0xffff);
    const int mis = (int)(((uintptr_t)codes + (uintptr_t)g0) & 3);
    for (int i = threadIdx.x; i < (mis + bytes + 3) / 4; i += NT) ((uint32_t*)buf)[i] = kPadCode * 0x01010101u;
    __syncthreads();
    int j = excl >> 16, r = excl & 0xffff;  // fragment starts and residues of the chunk before this thread's codons
#pragma unroll
    for (int k = 0; k < kTrPer; ++k) {
      if (!((live >> k) & 1u)) continue;
      if ((first >> k) & 1u) {
        const int64_t f = cf + j;
        const int64_t pos = g0 + kPadLen * (j + 1) + r;
        if (f < n_frags && pos < n_padded) {
          seq_start[f] = pos;
          frag[3 * f] = s / 6;
          frag[3 * f + 1] = S.frame;
          frag[3 * f + 2] = (int32_t)(i0 + k);
        }
        ++j;
      }
      buf[mis + kPadLen * j + r] = (uint8_t)(c[k / 4] >> (8 * (k % 4)));
      ++r;
    }
    __syncthreads();
    // whole dwords, and the bytes at either end that share one with other chunks
    const int n = (int)min((int64_t)bytes, max(n_padded - g0, (int64_t)0));
    uint8_t* dst = codes + g0 - mis;
    for (int i = threadIdx.x; 4 * i < mis + n; i += NT) {
      if (4 * i >= mis && 4 * i + 4 <= mis + n) {
        ((uint32_t*)dst)[i] = ((const uint32_t*)buf)[i];
      } else {
        for (int b = max(4 * i, mis); b < min(4 * i + 4, mis + n); ++b) dst[b] = buf[b];
      }
    }
    cf += tot >> 16;
    cr += tot & 0xffff;
    __syncthreads();
  }
}

struct TrWs {
  TrHeader* hdr;
  int32_t* err;  // hdr->err
  int64_t* nfrag;
  int64_t* nres;
};

TrWs tr_carve(void* d_ws, int32_t n_dna) {
  uint8_t* p = (uint8_t*)d_ws;
  TrWs W;
  W.hdr = (TrHeader*)p;
  W.err = &W.hdr->err;
  W.nfrag = (int64_t*)(p + 256);
  W.nres = (int64_t*)(p + 256 + align_up(sizeof(int64_t) * (6 * (size_t)n_dna + 1), 256));
  return W;
}

}  // namespace

size_t translate_ws_bytes(int32_t n_dna) {
  return 256 + 2 * align_up(sizeof(int64_t) * (6 * (size_t)n_dna + 1), 256);
}

int translate_count_impl(const uint8_t* d_dna, const int64_t* d_dna_start, int32_t n_dna, int64_t n_nt, void* d_ws,
                         int64_t* h_n_frags, int64_t* h_n_padded, hipStream_t s) {
  TrWs W = tr_carve(d_ws, n_dna);
  const CodonTable T = codon_table();
  const int streams = 6 * n_dna;
  const dim3 grid((unsigned)(streams > 0 ? streams : 1));
  hipLaunchKernelGGL(k_tr_clear, dim3(1), dim3(64), 0, s, W.err);
  if (streams > 0) {
    if (n_nt <= (int64_t)n_dna * kTrShortNt)
      hipLaunchKernelGGL(k_tr_count<kTrShort>, grid, dim3(kTrShort), 0, s, d_dna, d_dna_start, n_dna, n_nt, T, W.nfrag,
                         W.nres, W.err);
    else
      hipLaunchKernelGGL(k_tr_count<kTrLong>, grid, dim3(kTrLong), 0, s, d_dna, d_dna_start, n_dna, n_nt, T, W.nfrag,
                         W.nres, W.err);
  }
  // one workgroup scans up to 4096 streams in 4 steps; the parts' sums cost a launch
  const int parts = streams > 4 * kTrScanThreads ? kScanParts : 1;
  if (parts > 1)
    hipLaunchKernelGGL(k_tr_part, dim3(parts), dim3(kTrScanThreads), 0, s, (const int64_t*)W.nfrag,
                       (const int64_t*)W.nres, streams, parts, W.hdr);
  hipLaunchKernelGGL(k_tr_scan, dim3(parts), dim3(kTrScanThreads), 0, s, W.nfrag, W.nres, streams, parts, W.hdr);
  PLAST_HIP(hipGetLastError());
  TrHeader h;
  PLAST_HIP(hipMemcpyAsync(&h, W.hdr, offsetof(TrHeader, part), hipMemcpyDeviceToHost, s));
  PLAST_HIP(hipStreamSynchronize(s));
  const int32_t err = h.err;
  const int64_t tf = h.frags, tr = h.res;
  if (err & 1) return set_error(PLAST_E_LAYOUT, "dna_start is not ascending within [0, n_nt]");
  if (err & 2) return set_error(PLAST_E_ALPHABET, "a nucleotide code is > 3");
  *h_n_frags = tf;
  *h_n_padded = (int64_t)kPadLen * (tf + 1) + tr;
  return PLAST_OK;
}

int translate_write_impl(const uint8_t* d_dna, const int64_t* d_dna_start, int32_t n_dna, int64_t n_nt, void* d_ws,
                         uint8_t* d_codes, int64_t n_padded, int64_t* d_seq_start, int32_t* d_frag, int64_t n_frags,
                         hipStream_t s) {
  TrWs W = tr_carve(d_ws, n_dna);
  const CodonTable T = codon_table();
  const dim3 grid((unsigned)(n_dna > 0 ? 6 * n_dna : 1));
  if (n_dna <= 0)
    hipLaunchKernelGGL(k_tr_pad, grid, dim3(256), 0, s, d_codes, n_padded, d_seq_start, n_frags);
  else if (n_nt <= (int64_t)n_dna * kTrShortNt)
    hipLaunchKernelGGL(k_tr_write<kTrShort>, grid, dim3(kTrShort), 0, s, d_dna, d_dna_start, n_dna, n_nt, T,
                       (const int64_t*)W.nfrag, (const int64_t*)W.nres, d_codes, n_padded, d_seq_start, d_frag,
                       n_frags, W.err);
  else
    hipLaunchKernelGGL(k_tr_write<kTrLong>, grid, dim3(kTrLong), 0, s, d_dna, d_dna_start, n_dna, n_nt, T,
                       (const int64_t*)W.nfrag, (const int64_t*)W.nres, d_codes, n_padded, d_seq_start, d_frag,
                       n_frags, W.err);
  PLAST_HIP(hipGetLastError());
  return PLAST_OK;
}

}  // namespace plast
