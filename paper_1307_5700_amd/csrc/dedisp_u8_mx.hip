// Brute-force incoherent dedispersion (Sec. 2.2.2) of 8-bit filterbanks
// without cleaning on the matrix cores, in exact integers, for gfx950.
//
//   D[d][t] = sum_c x[c][t + s[d][c]],   x[c][t] in 0..255
//
// Within a group of 16 adjacent DMs and 16 adjacent channels, the delays
// differ from a common slope by a few samples only: once the channels of a
// cell are staged along the slope, a DM reads its channel q = 0..S-1 cells
// further on, and S is small (4 to 12 on the 20 MHz beams).  The sum over
// channels is then, for each shift s, the product of the staged samples
// [time][channel] with a matrix [channel][DM] that holds 1 where q = s.  One
// v_mfma_i32_16x16x64_i8 adds 64 channels' terms at one shift to 16 outputs
// of 16 DMs.  Samples enter as x - 128, a signed byte; the constant 128 C is
// added at the end.  The sums are integers below 2^24 in magnitude, so every
// order of the adds gives the bits of the other 8-bit kernels.
//
// Geometry.  A workgroup covers 32 DMs (two groups) and BT outputs.  Channels
// are taken in steps of four cells of 16; ns steps form one partial sum,
// aligned to its middle channel: seen from there, output t of DM d sits in
// column t + (its delay there) - (the group's least).  As the delays of 16
// DMs spread (66 samples at the ends of the 1024-channel beam with 0.2 DM
// steps), a DM's outputs are taken at an offset that makes them spread
// equally to both sides of the band's middle, and the 576 columns of a
// partial sum hold BT = 576 - spread outputs (508 there).
//
// Roles (16 waves).  Eight producer waves, two sets of four that take steps
// in turn, load a quarter's 16 channels (unaligned words along the slope),
// transpose 4 x 4 bytes at a time and write cells of 16 channels.  Eight
// consumer waves own 144 columns of a DM group each, as 9 tiles: column
// 9 m + j is row m of tile j.  With that stride, tile j at shift s reads the
// cells that tile j + 1 reads at shift s - 1, so shifts taken together share
// operand reads: 12 for the first four shifts of 9 tiles and 10 for each two
// after them, instead of 9 a shift (fewer than four are taken as four, an odd
// one as two).  The odd stride spreads one quarter's reads over all banks.  At
// the end of a partial sum the columns go through LDS, and each wave adds four
// DMs' rows, each from its own offset, to 32-bit sums in registers.  Two staged
// steps alternate, one barrier per step.
//
// What bounds it (counters on the 1024-channel x 65536-sample x 640-DM beam):
// no one unit.  A step has 161 products of 16 clocks and 560 other vector
// instructions of 2.6 a SIMD, which hardly overlap (a probe: about one vector
// instruction per product): 36 % and 21 % of the cycles.  The LDS is busy for
// 60 % of them, half of that with bank conflicts (31 % of all cycles): a
// producer lane writes its 16 bytes 64 bytes from the next lane's, so lanes
// four apart meet, and an operand read spans four quarters whose first cells
// differ by any amount.  Few waves hide the rest, waits for LDS and barriers.
// 0.46 to 0.49 ms (0.52 on uniformly random bytes) against 1.75 ms for the
// packed 16-bit add kernel, 80 against 22 x 10^12 adds/s; 4096 channels x 1024
// DMs: 1.75 against 9.83 ms; 512 channels x 320 DMs x 16384 samples: 0.067
// against 0.134 ms.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "internal.h"
#include "tile_map.h"

namespace mbtp {
namespace {

constexpr int kJ = kMxJ, kGroups = kMxGroups, kBD = kMxBD, kW = kMxW, kCells = kMxCells;
constexpr int kPieces = kMxPieces;
constexpr int kPitch = kW + 4;                 // words of one row of partial sums
constexpr int kCons = kGroups * kPieces;       // consumer waves
constexpr int kProd = 8;                       // producer waves: two sets of four
constexpr int kWaves = kCons + kProd;
constexpr int kRows = kBD / kCons;             // output rows a consumer wave keeps
constexpr int kSegs = kMxMaxBT / 64;           // 64-output segments of a row
constexpr int kCW = kMxCW, kCS = 4 * kCW;      // channels of a cell, of a step
constexpr int kBufBytes = 4 * kCells * kCW;    // one staged step
constexpr int kPartWords = kBD * kPitch + 512; // a row is read up to 512 words past its offset
constexpr int kHold = 4;                       // shifts whose operands are made at once
static_assert(kPitch % 8 == 4, "rows an odd multiple of 16 bytes apart: conflict-free 16-byte writes");
static_assert(kJ % 2 == 1, "odd column stride: conflict-free operand reads");
static_assert(kCW == 16 && kCells % 4 == 0, "a cell is one 16-byte operand; four cells per producer lane");
static_assert(2 * kBufBytes + 4 * kPartWords == kMxLds, "LDS size");

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Pointers to global memory formed from integers: the address space is named,
// so that the loads are global and not generic ones, which also count as LDS
// operations.
template <typename T> using GlobalPtr = const __attribute__((address_space(1))) T*;
struct __attribute__((packed)) Word { uint32_t v; };     // at any byte

// Lane l's 64-bit value as a uniform pointer.
__device__ inline GlobalPtr<uint8_t> lane_ptr(uint64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
  return reinterpret_cast<GlobalPtr<uint8_t>>(((uint64_t)hi << 32) | lo);
}

// A channel's shift q (0..7) is held as the byte 1 << q: the operand for
// shift s holds 1 in the channels whose bit s is set.
__device__ inline i32x4 one_hot(uint4 m, int s) {
  const uint4 r = make_uint4((m.x >> s) & 0x01010101u, (m.y >> s) & 0x01010101u, (m.z >> s) & 0x01010101u,
                             (m.w >> s) & 0x01010101u);
  return __builtin_bit_cast(i32x4, r);
}

// The 9 tiles of a wave for SC consecutive shifts: cell u of a lane's columns
// is tile j's operand at shift u - j.  Two reads are in flight; the order is
// fixed (the scheduler would gather all reads first and spill).
template <int SC>
__device__ __forceinline__ void mma_shifts(i32x4 (&c)[kJ], const char* base, const i32x4* hot) {
  constexpr int N = kJ + SC - 1, D = 2;
  i32x4 f[D];
#pragma unroll
  for (int u = 0; u < D; ++u) f[u] = *reinterpret_cast<const i32x4*>(base + kCW * u);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      const int j = u - s;
      if (j >= 0 && j < kJ) c[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[u % D], hot[s], c[j], 0, 0, 0);
    }
    if (u + D < N) f[u % D] = *reinterpret_cast<const i32x4*>(base + kCW * (u + D));
  }
  __builtin_amdgcn_sched_barrier(0);
}

// First channel of quarter o of step st of partial sum sub: ns steps of four
// cells around a reference in their middle.  The outermost cells share a
// step, so that a step's cells need about the same number of shifts.
__device__ inline int cell_channel(int sub, int st, int o, int ns) {
  const int i = o < 2 ? 2 * st + o : 4 * ns - 2 * st - 4 + o;
  return (4 * ns * sub + i) * kCW;
}

// Counts steps as (partial sum, step of it), stopping at the last one.
struct StepCount {
  int sub = 0, st = 0, k = 0;
  __device__ void next(int ns, int nstep) {
    if (k + 1 >= nstep) return;
    ++k;
    if (++st == ns) st = 0, ++sub;
  }
};

// Ends the consumers' step k (-1: the first staging).  Partial sums of one
// step have a barrier of their own between collecting one and writing the
// next; every wave passes it.
__device__ __forceinline__ void end_step(const MxTables& T, int k) {
  if (T.ns == 1 && k >= 1) __syncthreads();
  __syncthreads();
}

// Stages one quarter (16 channels) of every other step.  A set's loads are
// in flight while the other set's step is written.
__device__ __forceinline__ void produce(const DedispArgs& A, const MxTables& T, int blk, int64_t T0, char* bufs,
                                        int lane, int pw) {
  constexpr int NPASS = (kCells + 255) / 256;    // four cells a lane and pass
  const int set = pw >> 2, qo = pw & 3;
  const int nstep = T.nsub * T.ns, C = A.C, L = (int)A.L;
  const int32_t* sb = T.sbase + (int64_t)blk * T.cpad + qo * kCW;
  const uint8_t* const xin = static_cast<const uint8_t*>(A.x);
  StepCount nx;                                  // the set's next step
  if (set == 1) nx.next(T.ns, nstep);
  uint32_t raw[NPASS][16];
  int base_l = sb[nx.k * kCS + (lane & 15)];     // lane i < 16: window start of channel i
  int cur_l = 0, left = 0;                       // of the loaded step: its base_l, channels that exist
  bool whole = true;                             // all its samples exist
  auto issue = [&] {
    const int ch0 = cell_channel(nx.sub, nx.st, qo, T.ns);
    const int64_t bl = T0 + base_l;
    const uint64_t at = reinterpret_cast<uint64_t>(xin) + (int64_t)min(ch0 + (lane & 15), C - 1) * A.ld;
    cur_l = base_l;
    left = C - ch0;
    nx.next(T.ns, nstep);
    nx.next(T.ns, nstep);
    base_l = sb[nx.k * kCS + (lane & 15)];
    whole = __builtin_amdgcn_ballot_w64(!(bl >= 0 && bl + NPASS * 256 <= L)) == 0 && left >= 16;
    if (whole) {
      const uint64_t from = at + bl;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const GlobalPtr<uint8_t> row = lane_ptr(from, i);
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
          raw[p][i] = reinterpret_cast<GlobalPtr<Word>>(row + (uint32_t)(256 * p + 4 * lane))->v;
      }
    } else {
      // at the chunk's ends the word nearest to the lane's samples, moved to
      // their place when it is written (rows are at least 4 bytes long)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const GlobalPtr<uint8_t> row = lane_ptr(at, i);
        const int r0 = (int)T0 + __builtin_amdgcn_readlane(cur_l, i) + 4 * lane;
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
          raw[p][i] = reinterpret_cast<GlobalPtr<Word>>(row + (uint32_t)max(min(r0 + 256 * p, L - 4), 0))->v;
        asm volatile("" ::: "memory");           // keeps the two paths' loads apart
      }
    }
  };
  auto emit = [&](int k) {
    if (!whole) {
      // samples outside the chunk (which no output reads) become 0, channels
      // past the last 0 after the bias
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r0 = (int)T0 + __builtin_amdgcn_readlane(cur_l, i) + 4 * lane;
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
          const int t = r0 + 256 * p, d = t - max(min(t, L - 4), 0);       // samples past the word loaded
          const uint32_t w = raw[p][i];
          const uint32_t v = d >= 0 ? (d < 4 ? w >> (8 * d) : 0u) : (d > -4 ? w << (-8 * d) : 0u);
          raw[p][i] = i < left ? v : 0x80808080u;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    char* dst = bufs + (k & 1) * kBufBytes + qo * (kCells * kCW) + 64 * lane;
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
      uint32_t cell[4][4];
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = raw[p][i + e] ^ 0x80808080u;      // x - 128
        const uint32_t t0 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u);
        const uint32_t t1 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
        const uint32_t t2 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);
        const uint32_t t3 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
        cell[0][i / 4] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
        cell[1][i / 4] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
        cell[2][i / 4] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
        cell[3][i / 4] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
      }
      if (256 * p + 4 * lane < kCells) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<uint4*>(dst + 256 * kCW * p + kCW * e) =
              make_uint4(cell[e][0], cell[e][1], cell[e][2], cell[e][3]);
      }
    }
  };
  if (set == 1) end_step(T, -1);
  issue();
#pragma unroll 1
  for (int k = set; k < nstep; k += 2) {
    emit(k);
    end_step(T, k - 1);
    issue();
    if (k + 1 < nstep) end_step(T, k);
  }
  end_step(T, nstep - 1);
}

__global__ __launch_bounds__(64 * kWaves) void dedisp_u8_mx_kernel(DedispArgs A, MxTables T) {
  extern __shared__ char lds[];
  char* const bufs = lds;
  int* const part = reinterpret_cast<int*>(lds + 2 * kBufBytes);
  const TileIdx ti = xcd_tile(blockIdx.x, A.n_dblocks, A.n_ttiles, A.ndms % kBD != 0);
  const int blk = ti.dblock;
  const int64_t T0 = (int64_t)ti.ttile * T.BT;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= kCons) {
    produce(A, T, blk, T0, bufs, lane, wave - kCons);
    return;
  }

  // ---- consumers: wave = (DM group g, columns pc * 144 .. of the partial sum)
  const int o = lane >> 4, dn = lane & 15;       // quarter; column row or DM of the group
  const int nstep = T.nsub * T.ns;
  const int g = wave / kPieces, pc = wave % kPieces;
  const char* hdr = reinterpret_cast<const char*>(T.hdr + ((int64_t)blk * nstep * kGroups + g) * 4);
  const char* hot = reinterpret_cast<const char*>(T.hot) + ((int64_t)blk * nstep * kGroups + g) * (64 * kCW);
  const char* po = reinterpret_cast<const char*>(T.poff + (int64_t)blk * T.nsub * kBD + wave * kRows);
  // steps past the plan's last in the table hold the bits of shifts 8..15
  const int high = A.n_dblocks * nstep;
  auto load_hdr = [&](int k) {
    return *reinterpret_cast<const int2*>(hdr + (int64_t)k * (kGroups * 32) + (uint32_t)(8 * o));
  };
  auto load_hot = [&](int k) {
    return *reinterpret_cast<const uint4*>(hot + (int64_t)k * (kGroups * 64 * kCW) + (uint32_t)(lane * kCW));
  };
  auto load_po = [&](int b) {
    return *reinterpret_cast<const int*>(po + (int64_t)b * (kBD * 4) + (uint32_t)(4 * (lane & (kRows - 1))));
  };
  int acc[kRows][kSegs];
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int s = 0; s < kSegs; ++s) acc[r][s] = 0;
  i32x4 c[kJ];
  int2 hn = load_hdr(0);
  uint4 qn = load_hot(0);
  int pn = load_po(0), pcur = 0;
  const int col = dn * kJ + pc * (16 * kJ);      // first column of the lane's operand rows
  int* const pw = part + (g * 16 + dn) * kPitch + pc * (16 * kJ) + o * (4 * kJ);

  // Adds the partial sum's rows of this wave's four DMs, each from its own
  // column on (two rows' reads in flight together).
  auto read_part = [&] {
#pragma unroll
    for (int r = 0; r < kRows; r += 2) {
      int v[2][kSegs];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int* row = part + (wave * kRows + r + q) * kPitch + __builtin_amdgcn_readlane(pcur, r + q) + lane;
#pragma unroll
        for (int s = 0; s < kSegs; ++s) v[q][s] = row[64 * s];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int s = 0; s < kSegs; ++s) acc[r + q][s] += v[q][s];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Writes the wave's columns: a lane holds DM dn's columns 36 o + 9 i + j of
  // the piece in element i of tile j, 36 consecutive words of its row.
  auto write_part = [&] {
#pragma unroll
    for (int k = 0; k < kJ; ++k) {
      i32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = c[(4 * k + e) % kJ][(4 * k + e) / kJ];
      *reinterpret_cast<i32x4*>(pw + 4 * k) = w;
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  __syncthreads();
  int cur = 0, k = 0;
#pragma unroll 1
  for (int sub = 0; sub < T.nsub; ++sub) {
    // The previous partial sum is collected during the first step of this
    // one, by one DM group before its products and by the other after them:
    // the LDS reads of the one overlap the products of the other.  The
    // barrier that ends the step lies between these reads and the next
    // writes; with one step per partial sum, one before the writes does.
    if (sub > 0 && g == 0) read_part();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kJ; ++j) c[j] = i32x4{0, 0, 0, 0};
#pragma unroll 1
    for (int st = 0; st < T.ns; ++st, ++k) {
      const int S = __builtin_amdgcn_readfirstlane(hn.y);
      const char* base = bufs + cur * kBufBytes + kCW * (o * kCells + hn.x + col);
      const uint4 q = qn;
      const int kn = min(k + 1, nstep - 1);
      hn = load_hdr(kn);
      qn = load_hot(kn);
      uint4 qh = q;
      if (S > 8) qh = load_hot(high + k);
      i32x4 h[kHold];
#pragma unroll
      for (int s = 0; s < kHold; ++s) h[s] = one_hot(q, s);
      mma_shifts<kHold>(c, base, h);
#pragma unroll 1
      for (int s0 = kHold; s0 < S; s0 += 2) {
        const uint4 m = s0 < 8 ? q : qh;
        const i32x4 h2[2] = {one_hot(m, s0 & 7), one_hot(m, (s0 & 7) + 1)};
        mma_shifts<2>(c, base + kCW * s0, h2);
      }
      if (st == 0) {
        if (sub > 0 && g != 0) read_part();
        pcur = pn;
        pn = load_po(min(sub + 1, T.nsub - 1));
      }
      if (T.ns == 1 && k >= 1) __syncthreads();
      if (st == T.ns - 1) write_part();
      __syncthreads();
      cur ^= 1;
    }
  }
  read_part();

  // ---- store: column y of DM d is output T0 + y - moff[d] ----
  int ln = lane;
  asm volatile("" : "+v"(ln));                   // keeps the addresses out of the loop above
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int d = blk * kBD + wave * kRows + r;
    if (d >= A.ndms) continue;
    const int64_t t1 = T0 - __builtin_amdgcn_readfirstlane(T.moff[d]);
    float* orow = A.out + (int64_t)d * A.ld_out;
#pragma unroll
    for (int s = 0; s < kSegs; ++s) {
      const int y = 64 * s + ln;
      const int64_t t = t1 + y;
      if (y < T.BT && t >= 0 && t < A.nout) orow[t] = (float)(acc[r][s] + 128 * A.C);
    }
  }
}

// Statistics and, where there is room for them, tables of one plan: one
// workgroup per (partial sum, DM block).
__global__ __launch_bounds__(256) void mx_setup_kernel(MxSetup P) {
  const int sub = blockIdx.x, blk = blockIdx.y, tid = threadIdx.x;
  const int C = P.C, ns = P.ns, G = ns * kCS, nstep = P.nsub * ns, ncell = 4 * ns;
  const bool tables = P.hdr != nullptr;
  const int d0 = blk * kBD, dc = d0 + min(kBD, P.ndms - d0) / 2;       // the block's middle DM
  const int mid = C / 2, ref = min(sub * G + G / 2, C - 1);
  constexpr int kNone = 0x3fffffff;
  __shared__ int m[kBD], e[kBD], mlo, mhi, emin[kGroups], spread[kGroups], need;
  __shared__ int lo[4 * kMxMaxSteps], amin[4 * kMxMaxSteps][kGroups], amax[4 * kMxMaxSteps][kGroups];
  // rows past the plan's last repeat it
  auto del = [&](int d, int c) { return P.delays[(int64_t)min(d, P.ndms - 1) * C + c]; };
  if (tid < ncell) {
    lo[tid] = kNone;
    for (int g = 0; g < kGroups; ++g) amin[tid][g] = kNone, amax[tid][g] = -kNone;
  }
  // m: a DM's outputs are taken m later than the tile's columns, so that its
  // delays at the band's middle equal the middle DM's; e: its column there
  if (tid < kBD) {
    m[tid] = del(d0 + tid, mid) - del(dc, mid);
    e[tid] = del(d0 + tid, ref) - m[tid];
  }
  __syncthreads();
  if (tid == 0) {
    mlo = mhi = m[0];
    for (int i = 1; i < kBD; ++i) mlo = min(mlo, m[i]), mhi = max(mhi, m[i]);
    for (int g = 0; g < kGroups; ++g) {
      int v = e[16 * g], w = v;
      for (int i = 1; i < 16; ++i) v = min(v, e[16 * g + i]), w = max(w, e[16 * g + i]);
      emin[g] = v;
      spread[g] = w - v;
    }
    need = 0;
  }
  __syncthreads();
  int ymin = emin[0];
  for (int g = 1; g < kGroups; ++g) ymin = min(ymin, emin[g]);
  // delay relative to the reference channel and to the middle DM
  auto rel = [&](int d, int c) { return (del(d, c) - del(d, ref)) - (del(dc, c) - del(dc, ref)); };
  for (int i = tid; i < ncell * kCW * kBD; i += 256) {
    const int d = i % kBD, cell = i / kBD / kCW, g = d / 16;
    const int c = cell_channel(sub, cell / 4, cell % 4, ns) + i / kBD % kCW;
    if (c < C) {
      const int q = rel(d0 + d, c);
      atomicMin(&lo[cell], q);
      atomicMin(&amin[cell][g], q);
      atomicMax(&amax[cell][g], q);
    }
  }
  __syncthreads();
  // a cell is staged from its block's least shift on; a group starts
  // amin - lo cells later and needs S shifts, the most of the step's cells
  for (int i = tid; i < ns * kGroups; i += 256) {
    const int st = i / kGroups, g = i % kGroups;
    int S = 1;
    for (int cell = 4 * st; cell < 4 * st + 4; ++cell)
      if (lo[cell] < kNone) S = max(S, amax[cell][g] - amin[cell][g] + 1);
    for (int q = 0; q < 4; ++q) {
      const int cell = 4 * st + q;
      const int off = emin[g] - ymin + (lo[cell] < kNone ? amin[cell][g] - lo[cell] : 0);
      if (tables) P.hdr[(((int64_t)blk * nstep + sub * ns + st) * kGroups + g) * 4 + q] = make_int2(off, S);
      atomicMax(&need, off + spread[g] + S);
    }
    atomicMax(&P.stats[2], S);
  }
  for (int i = tid; tables && i < G; i += 256) {
    const int cell = i / kCW;
    const int c = min(cell_channel(sub, cell / 4, cell % 4, ns) + i % kCW, C - 1);
    P.sbase[(int64_t)blk * P.cpad + sub * G + i] =
        mlo + ymin + (del(dc, c) - del(dc, ref)) + (lo[cell] < kNone ? lo[cell] : 0);
  }
  const int64_t half = (int64_t)gridDim.y * nstep * kGroups * 64 * kCW;
  for (int i = tid; tables && i < ns * kGroups * 64 * kCW; i += 256) {
    const int ch = i % kCW, lane = (i / kCW) % 64, g = (i / kCW / 64) % kGroups, st = i / kCW / 64 / kGroups;
    const int cell = 4 * st + (lane >> 4), c = cell_channel(sub, st, lane >> 4, ns) + ch;
    const int q = c < C ? rel(d0 + 16 * g + (lane & 15), c) - amin[cell][g] : -1;
    uint8_t* h = P.hot + ((((int64_t)blk * nstep + sub * ns + st) * kGroups + g) * 64 + lane) * kCW + ch;
    h[0] = q >= 0 && q < 8 ? (uint8_t)(1 << q) : 0;
    h[half] = q >= 8 && q < 16 ? (uint8_t)(1 << (q - 8)) : 0;
  }
  if (tid < kBD) {
    const int po = e[tid] - emin[tid / 16];
    if (tables) P.poff[((int64_t)blk * P.nsub + sub) * kBD + tid] = po;
    atomicMax(&P.stats[0], po);
    if (sub == 0) {
      if (tables) P.moff[d0 + tid] = m[tid] - mlo;
      atomicMax(&P.stats[3], mhi - mlo);
    }
  }
  __syncthreads();
  if (tid == 0) atomicMax(&P.stats[1], need);
}

__global__ void mx_clear_kernel(int32_t* stats) {
  if (threadIdx.x < 4) stats[threadIdx.x] = 0;
}

}  // namespace

hipError_t dedisp_u8_mx_prepare() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(dedisp_u8_mx_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kMxLds);
}

hipError_t launch_mx_setup(const MxSetup& p, int nblk, hipStream_t s) {
  hipLaunchKernelGGL(mx_clear_kernel, dim3(1), dim3(64), 0, s, p.stats);
  hipLaunchKernelGGL(mx_setup_kernel, dim3((unsigned)p.nsub, (unsigned)nblk), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_dedisp_u8_mx(const DedispArgs& a, const MxTables& t, hipStream_t s) {
  const unsigned grid = (unsigned)a.n_dblocks * (unsigned)a.n_ttiles;
  hipLaunchKernelGGL(dedisp_u8_mx_kernel, dim3(grid), dim3(64 * kWaves), kMxLds, s, a, t);
  return hipGetLastError();
}

}  // namespace mbtp
