// Particle kernels of the compressed PM step for gfx950: integer CIC deposit, the two move passes
// (count, then encode + scatter), the per-cell link/scan/statistics kernels, the initial-condition
// lattice move and the load path.
//
// Storage (Sec. 2.1-2.2): particles are cell ordered; position codes chi (Eq. (chi)) and velocity
// codes nu (Eq. (nu)) are packed into words of two or three planes (Codes below); per coarse cell the
// count, the storage offset, the mean velocity v_c and the decode scale sigma sqrt(2/pi) of Eq. (v).
//
// All kernels work on tiles of T^3 coarse cells (one workgroup per tile). Deposit gathers: the
// workgroup that owns a tile of fine cells reads the particles of its tile and of the ring of
// neighbouring coarse cells and accumulates exact integer CIC weights in LDS (no float atomics,
// no global atomics), so the density is bit-reproducible. The move passes scatter: each particle
// is handled by the workgroup that owns its coarse cell; the potential tile with a 3-cell halo
// sits in LDS for the 4-point gradient.
//
// The arithmetic follows one fixed sequence of IEEE operations so that the encoding, cell counts
// and order are reproducible bit for bit from identical inputs: the compiler forms no fused
// multiply-adds of its own (-ffp-contract=off), and the fused ones the sequence names -- velocity
// decode, the interpolation lerps, kick and drift -- are written out as fmaf.
#include <cstring>
#include <type_traits>


#include "cube_internal.h"
#include "launch_groups.h"

namespace cube {
namespace {

constexpr int T = 4;            // coarse cells per tile side
// tile offsets (x, y, z) of own cell s (x fastest), by shifts: s is never negative
__device__ __forceinline__ void tile_xyz(int s, int& ox, int& oy, int& oz) {
  static_assert(T == 4, "shifts assume four cells per side");
  const unsigned u = (unsigned)s;
  ox = (int)(u & 3u);
  oy = (int)((u >> 2) & 3u);
  oz = (int)(u >> 4);
}
constexpr int TC = T * T * T;   // own cells per tile
constexpr int F = 4 * T;        // fine cells per tile side
constexpr int PH = F + 6;       // potential tile side (3-cell halo)
constexpr int RG = T + 2;       // new-cell region side (tile + ring)
constexpr int RC = RG * RG * RG;
constexpr int LINK_BLK = 256;

template <int NCHI>
using chi_t = std::conditional_t<NCHI == 1, uint8_t, uint16_t>;
template <int NNU>
using nu_t = std::conditional_t<NNU == 1, int8_t, int16_t>;

// The codes of one particle as they lie in memory. The first plane's word (4 bytes with 1-byte
// positions, 8 with 2-byte ones) holds the three position codes and fills up with velocity codes;
// the rest of these follow in planes of 4, 2 or 1 bytes:
//   x1v1  [chi0 chi1 chi2 nu0] [nu1 nu2]            x1v2  [chi0 chi1 chi2 nu0lo] [nu1 nu2] [nu0hi]
//   x2v1  [chi0 chi1 chi2 nu0 nu1] [nu2]            x2v2  [chi0 chi1 chi2 nu0] [nu1 nu2]
// that is 3 (n_chi + n_nu) bytes a particle in all, each plane `cap` words long and aligned to its
// word. A plane per code cost six byte loads and six byte stores a particle, and each store
// instruction of a scatter makes one request per destination line (about a dozen), which bounded it.
// With 512^3 x1v1 particles: scatter 1340 -> 990 us, deposit, which reads the first plane only, 1436 ->
// 1075 us early and 1793 -> 1369 us clustered.
template <int NCHI, int NNU>
struct Codes {
  uint32_t a0, a1, b, c;  // first plane (a1: 2-byte positions), second, third

  __device__ __forceinline__ void load_chi(const void* base, int64_t p) {
    if constexpr (NCHI == 1) {
      a0 = static_cast<const uint32_t*>(base)[p];
    } else {
      const uint2 w = static_cast<const uint2*>(base)[p];
      a0 = w.x;
      a1 = w.y;
    }
  }
  __device__ __forceinline__ void load(const void* base, int64_t cap, int64_t p) {
    load_chi(base, p);
    const char* const rest = static_cast<const char*>(base) + cap * (NCHI == 1 ? 4 : 8);
    if constexpr (NCHI == 1 && NNU == 1) b = reinterpret_cast<const uint16_t*>(rest)[p];
    if constexpr (NNU == 2) b = reinterpret_cast<const uint32_t*>(rest)[p];
    if constexpr (NCHI == 1 && NNU == 2) c = reinterpret_cast<const uint8_t*>(rest + cap * 4)[p];
    if constexpr (NCHI == 2 && NNU == 1) c = reinterpret_cast<const uint8_t*>(rest)[p];
  }
  __device__ __forceinline__ void store(void* base, int64_t cap, int64_t p) const {
    if constexpr (NCHI == 1) static_cast<uint32_t*>(base)[p] = a0;
    else static_cast<uint2*>(base)[p] = make_uint2(a0, a1);
    char* const rest = static_cast<char*>(base) + cap * (NCHI == 1 ? 4 : 8);
    if constexpr (NCHI == 1 && NNU == 1) reinterpret_cast<uint16_t*>(rest)[p] = (uint16_t)b;
    if constexpr (NNU == 2) reinterpret_cast<uint32_t*>(rest)[p] = b;
    if constexpr (NCHI == 1 && NNU == 2) reinterpret_cast<uint8_t*>(rest + cap * 4)[p] = (uint8_t)c;
    if constexpr (NCHI == 2 && NNU == 1) reinterpret_cast<uint8_t*>(rest)[p] = (uint8_t)c;
  }
  __device__ __forceinline__ void chi(int* ch) const {
    if constexpr (NCHI == 1) {
      ch[0] = (int)(a0 & 255u);
      ch[1] = (int)((a0 >> 8) & 255u);
      ch[2] = (int)((a0 >> 16) & 255u);
    } else {
      ch[0] = (int)(a0 & 65535u);
      ch[1] = (int)(a0 >> 16);
      ch[2] = (int)(a1 & 65535u);
    }
  }
  __device__ __forceinline__ void nu(int* n) const {
    const uint32_t t = (NCHI == 1 ? a0 >> 24 : a1 >> 16);  // what follows the positions in the first plane
    if constexpr (NNU == 1) {
      n[0] = (int)(int8_t)t;
      n[1] = (int)(int8_t)(NCHI == 1 ? b : t >> 8);
      n[2] = (int)(int8_t)(NCHI == 1 ? b >> 8 : c);
    } else {
      n[0] = (int)(int16_t)(NCHI == 1 ? t | (c << 8) : t);
      n[1] = (int)(int16_t)b;
      n[2] = (int)(int16_t)(b >> 16);
    }
  }
  // position codes already packed: chi0 | chi1 << 8 | chi2 << 16 in w, or chi0 | chi1 << 16 in w, chi2 in w2
  __device__ __forceinline__ void pack(uint32_t w, uint32_t w2, const int* n) {
    a0 = w;
    a1 = w2;
    if constexpr (NNU == 1) {
      const uint32_t n0 = (uint32_t)n[0] & 255u, n1 = (uint32_t)n[1] & 255u, n2 = (uint32_t)n[2] & 255u;
      if constexpr (NCHI == 1) {
        a0 |= n0 << 24;
        b = n1 | (n2 << 8);
      } else {
        a1 |= (n0 << 16) | (n1 << 24);
        c = n2;
      }
    } else {
      const uint32_t n0 = (uint32_t)n[0] & 65535u;
      b = ((uint32_t)n[1] & 65535u) | ((uint32_t)n[2] << 16);
      if constexpr (NCHI == 1) {
        a0 |= n0 << 24;
        c = n0 >> 8;
      } else {
        a1 |= n0 << 16;
      }
    }
  }
  __device__ __forceinline__ void set(const int* ch, const int* n) {
    if constexpr (NCHI == 1) pack((uint32_t)(ch[0] | (ch[1] << 8) | (ch[2] << 16)), 0u, n);
    else pack((uint32_t)ch[0] | ((uint32_t)ch[1] << 16), (uint32_t)ch[2], n);
  }
};

__device__ __forceinline__ int wrapi(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }

__device__ __forceinline__ void set_flag(uint32_t* flags, uint32_t f) { atomicOr(flags, f); }

// number of lanes below this one in the wave mask m
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A step whose error flags are set is not applied: the kernels that write the next state (link,
// scan, cell statistics, scatter) return at once, so the state stays the one before the failing
// step, and so it does through every later step enqueued behind it. The flag word is read once per
// workgroup (through LDS), so all of a workgroup's waves take the same branch even when another
// workgroup raises a flag meanwhile.
__device__ __forceinline__ bool workgroup_step_failed(const uint32_t* flags) {
  __shared__ uint32_t failed;
  if (threadIdx.x == 0) failed = __atomic_load_n(flags, __ATOMIC_RELAXED);
  __syncthreads();
  return failed != 0u;
}

// The deposit and the count pass of a phase enqueued behind a failed one find their state in the buffer
// that the failed phase left as it was (never written, or a new count beside an old offset): they must not
// follow it. flags[1], the failed phase's code, says so; it is written between phases only, so the
// workgroups of a launch agree. (flags[0] may be raised by the launch itself, whose other tiles still
// have to raise theirs: the most telling of the errors is the one reported.)
__device__ __forceinline__ bool earlier_phase_failed(const uint32_t* flags) { return flags[1] != 0u; }

// exclusive prefix of up to 256 uint32 values held one per thread; returns the total
__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* out, int n, uint32_t* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t x = (tid < n) ? v : 0u;
  uint32_t inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t wbase = 0, total = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    if (w < wave) wbase += wsum[w];
    total += wsum[w];
  }
  if (tid < n) out[tid] = wbase + inc - x;
  if (tid == 0) out[n] = total;
  __syncthreads();
  return total;
}

template <unsigned CTRL, unsigned ROWS = 0xF>
__device__ __forceinline__ unsigned long long dpp_add_u64(unsigned long long v) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  uint32_t l2, h2;
  if constexpr (ROWS == 0xF) {
    // every row written: lanes without a source read 0 (bound control), no old value needed
    l2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, CTRL, 0xF, 0xF, true);
    h2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, CTRL, 0xF, 0xF, true);
  } else {
    l2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, ROWS, 0xF, false);
    h2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, ROWS, 0xF, false);
  }
  unsigned int carry;
  const unsigned int rl = __builtin_addc(lo, l2, 0u, &carry);
  const unsigned int rh = __builtin_addc(hi, h2, carry, &carry);
  return ((unsigned long long)rh << 32) | rl;
}

// One step of the 64-bit inclusive scan: v += (v of the lane DPP selects, 0 where there is none;
// rows outside the row mask unchanged), as a carry-propagating add whose first operand is read
// through DPP. The s_nop before each step covers the two wait states a DPP read needs after a VALU
// write of the same register; the one after the block keeps later DPP reads of lo / hi safe.
#define CUBE_DPP_ADD64(lo, hi, CTRL, RMASK)                                                        \
  asm volatile("s_nop 1\n\t"                                                                     \
               "v_add_co_u32_dpp %0, vcc, %0, %0 " CTRL " row_mask:" RMASK                        \
               " bank_mask:0xf bound_ctrl:1\n\t"                                                 \
               "v_addc_co_u32_dpp %1, vcc, %1, %1, vcc " CTRL " row_mask:" RMASK                  \
               " bank_mask:0xf bound_ctrl:1\n\t"                                                 \
               "s_nop 1"                                                                          \
               : "+v"(lo), "+v"(hi)                                                               \
               :                                                                                  \
               : "vcc")

// inclusive prefix sum over the 64 lanes (every lane active): shifts by 1, 2, 4, 8 inside each
// row of 16 lanes, then the totals of rows 0 and 2 into rows 1 and 3, then that of rows 0-1 into
// rows 2 and 3
__device__ __forceinline__ unsigned long long wave_scan_u64(unsigned long long v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  CUBE_DPP_ADD64(lo, hi, "row_shr:1", "0xf");
  CUBE_DPP_ADD64(lo, hi, "row_shr:2", "0xf");
  CUBE_DPP_ADD64(lo, hi, "row_shr:4", "0xf");
  CUBE_DPP_ADD64(lo, hi, "row_shr:8", "0xf");
  CUBE_DPP_ADD64(lo, hi, "row_bcast:15", "0xa");
  CUBE_DPP_ADD64(lo, hi, "row_bcast:31", "0xc");
  return ((unsigned long long)hi << 32) | lo;
}

// the same for values whose sum is below 2^32
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

__device__ __forceinline__ unsigned long long read_lane_u64(unsigned long long v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}

// sum over the 64 lanes (every lane active), returned to all lanes
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
  v = dpp_add_u64<0xB1>(v);   // quad_perm [1,0,3,2]
  v = dpp_add_u64<0x4E>(v);   // quad_perm [2,3,0,1]
  v = dpp_add_u64<0x141>(v);  // row_half_mirror
  v = dpp_add_u64<0x140>(v);  // row_mirror: every lane holds its 16-lane row sum
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  unsigned long long t = 0;
#pragma unroll
  for (int r = 15; r < 64; r += 16)
    t += ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)hi, r) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)lo, r);
  return t;
}

// sum over the 64 lanes (every lane active), in all lanes
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);  // row_half_mirror
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);  // row_mirror: the 16-lane row's sum
  uint32_t t = 0;
#pragma unroll
  for (int r = 15; r < 64; r += 16) t += (uint32_t)__builtin_amdgcn_readlane((int)v, r);
  return t;
}
__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) { return wave_sum_u64(v); }

struct TileGeom {
  int cx0, cy0, cz0;
};
__device__ __forceinline__ TileGeom tile_of(int b, int nt) {
  TileGeom g;
  g.cx0 = (b % nt) * T;
  g.cy0 = ((b / nt) % nt) * T;
  g.cz0 = (b / (nt * nt)) * T;
  return g;
}

// ---------------------------------------------------------------------------------------------
// CIC deposit (Sec. 3 "CIC"; cell centres at i + 1/2), exact integer weights, gather by tile.
// ---------------------------------------------------------------------------------------------
struct DepArgs {
  const void* codes;
  const uint32_t* cnt;
  const uint64_t* off;
  int64_t cap;
  float* mesh;
  int64_t pitch_f;
  int nm, nc;
  int zc;  // coarse layers per z chunk
  double inv_mean;
  const uint32_t* flags;
};

constexpr int NSLOT = 6;  // fine planes a coarse layer can touch
constexpr int MANY = 12;  // lanes on one corner cell from which their weights are summed before the LDS add

// Streaming gather: the workgroup owns a column of DTX x DTX coarse cells (DF = 4 DTX fine cells a
// side) over the fine planes of coarse layers [cz0, cz1). It walks the source coarse layers
// cz0-1 .. cz1 in order, each time reading the particles of the DR x DR cells (column + ring), and adds
// exact integer CIC weights to a rolling set of NSLOT fine planes in LDS. After layer sz, planes up
// to 4 sz + 2 receive no more mass: those it owns are converted once to FP32 delta and written, and
// all their slots cleared.
//
// The planes in LDS have a border of one cell, so that the eight corners of a particle that reaches the
// column are added without a test: border cells and planes outside [4 cz0, 4 cz1) collect what nobody
// reads. A particle of the ring that reaches nothing is skipped by one comparison of its corner.
//
// Bound by vector issue where particles are spread (116 instructions per 64 particles of the column) and by
// LDS adds to one address where they cluster. With 512^3 particles on as many cells 1075 -> 685 us early
// and 1370 -> 986 clustered against columns with a tested corner each and 4 layers a chunk; 256^3 on
// 512^3 cells 412 -> 342. Where cells hold few particles the work per layer counts: the first wavefront alone
// reads and scans the layer's counts, and a thread converts the same column of fine cells in every plane
// (with all wavefronts scanning and the converted cells numbered anew 128^3 on 256^3 65 us, now 49; 96^3
// on 192^3 39 and 29; 256^3 on 512^3 375 and 342).
template <int DTX>
struct DepCfg {
  static constexpr int DF = 4 * DTX;
  static constexpr int DR = DTX + 2, DRC = DR * DR;
  static constexpr int PX = DF + 3, PLANE = PX * (DF + 2);  // bordered plane (an odd pitch spreads the banks)
};

template <int NCHI, int DTX, int BLK>
__device__ __forceinline__ void deposit_column(const DepArgs& a, const unsigned lb) {
  constexpr int SH = 8 * NCHI - 1;
  using C = DepCfg<DTX>;
  constexpr int DF = C::DF, DR = C::DR, DRC = C::DRC, PX = C::PX, PLANE = C::PLANE;
  static_assert(DRC <= 128, "source cells in two lane registers");
  __shared__ __align__(16) unsigned long long rho[NSLOT * PLANE];
  __shared__ uint32_t cbeg[(DRC > 64 ? DRC : 64) + 1];
  __shared__ uint64_t crel[DRC > 64 ? DRC : 64];
  __shared__ int corner[DRC];  // word of fine cell (0, 0) of a source cell in a bordered plane
  const bool failed = earlier_phase_failed(a.flags);  // requested first, tested before a code is read
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned ncol = (unsigned)(a.nc / DTX), cols = ncol * ncol;
  const unsigned bxy = lb % cols, bz = lb / cols;
  const int cx0 = (int)(bxy % ncol) * DTX, cy0 = (int)(bxy / ncol) * DTX;
  const int cz0 = (int)bz * a.zc;
  const int cz1 = min(cz0 + a.zc, a.nc);
  const int pz0 = 4 * cz0, pz1 = 4 * cz1;  // owned fine planes [pz0, pz1)
  for (int i = threadIdx.x; i < NSLOT * PLANE / 2; i += BLK) reinterpret_cast<uint4*>(rho)[i] = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x < DRC) corner[threadIdx.x] = ((int)threadIdx.x / DR * 4 - 3) * PX + ((int)threadIdx.x % DR * 4 - 3);
  // 32-bit accumulators where no sum can reach 2^32: a fine cell receives mass only from particles of
  // the 2^3 coarse cells around it, each weighing 2^(3 SH) in total, so with 1-byte codes 2047 particles
  // in every such block of the workgroup's source cells are few enough
  __shared__ uint32_t smax;
  if (threadIdx.x == 0) smax = 0u;
  __syncthreads();
  if constexpr (NCHI == 1) {
    const int nb = (DR - 1) * (DR - 1) * (cz1 - cz0 + 1);
    uint32_t m = 0u;
    for (int i = threadIdx.x; i < nb; i += BLK) {
      const int bx = i % (DR - 1), by = (i / (DR - 1)) % (DR - 1), bzz = i / ((DR - 1) * (DR - 1));
      uint32_t n = 0u;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t c = (uint32_t)wrapi(cx0 - 1 + bx + (j & 1), a.nc) +
                           (uint32_t)a.nc * ((uint32_t)wrapi(cy0 - 1 + by + ((j >> 1) & 1), a.nc) +
                                             (uint32_t)a.nc * (uint32_t)wrapi(cz0 - 1 + bzz + (j >> 2), a.nc));
        n += min(a.cnt[c], 4096u);
      }
      m = max(m, n);
    }
    if (m > 2047u) atomicMax(&smax, m);
  }
  __syncthreads();
  if (failed) return;
  const bool narrow = NCHI == 1 && (uint32_t)__builtin_amdgcn_readfirstlane((int)smax) <= 2047u;
  // the layer's source cells, in the lanes of the first wavefront: cells 0 .. 63 and 64 .. DRC - 1
  __shared__ uint32_t layer[2];  // particles of the layer, and whether lanes will share cells
  uint32_t cnt_n[2];
  uint64_t off_n[2];
  auto request = [&](int sz) {
    const int gz = wrapi(sz, a.nc);
#pragma unroll
    for (int h = 0; h < (DRC > 64 ? 2 : 1); ++h) {
      const int t = lane + 64 * h;
      cnt_n[h] = 0u;
      off_n[h] = 0u;
      if (t < DRC) {
        const uint32_t c = (uint32_t)wrapi(cx0 + t % DR - 1, a.nc) +
                           (uint32_t)a.nc * ((uint32_t)wrapi(cy0 + t / DR - 1, a.nc) + (uint32_t)a.nc * (uint32_t)gz);
        cnt_n[h] = a.cnt[c];
        off_n[h] = a.off[c];
      }
    }
  };
  // this thread's column of fine cells, in a bordered plane and in a plane of the mesh
  const int mine = ((int)threadIdx.x / DF + 1) * PX + (int)threadIdx.x % DF + 1;
  const uint32_t out = (uint32_t)(4 * cy0 + (int)threadIdx.x / DF) * (uint32_t)a.pitch_f + (uint32_t)(4 * cx0 + (int)threadIdx.x % DF);
  if (wave == 0) request(cz0 - 1);
  uint32_t* const rho32 = reinterpret_cast<uint32_t*>(rho);
  int first = ((4 * (cz0 - 1) - 1) % NSLOT + NSLOT) % NSLOT;  // slot of plane 4 sz - 1
  for (int sz = cz0 - 1; sz <= cz1; ++sz, first = first + 4 >= NSLOT ? first + 4 - NSLOT : first + 4) {
    if (wave == 0) {
      uint32_t inc[2];
      inc[0] = wave_scan_u32(cnt_n[0]);
      uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)inc[0], 63);
      if constexpr (DRC > 64) {
        inc[1] = n + wave_scan_u32(cnt_n[1]);
        n = (uint32_t)__builtin_amdgcn_readlane((int)inc[1], 63);
      }
      cbeg[lane] = inc[0] - cnt_n[0];
      crel[lane] = off_n[0] - (inc[0] - cnt_n[0]);
      if (DRC > 64 && lane + 64 < DRC) {
        cbeg[lane + 64] = inc[1] - cnt_n[1];
        crel[lane + 64] = off_n[1] - (inc[1] - cnt_n[1]);
      }
      // lanes share a cell where it holds a good part of the layer's particles
      bool crowd = __ballot((uint64_t)cnt_n[0] * 64u >= (uint64_t)MANY * n) != 0ull;
      if constexpr (DRC > 64) crowd |= __ballot((uint64_t)cnt_n[1] * 64u >= (uint64_t)MANY * n) != 0ull;
      if (lane == 0) {
        cbeg[DRC] = n;
        layer[0] = n;
        layer[1] = crowd ? 1u : 0u;
      }
      if (sz < cz1) request(sz + 1);
    }
    __syncthreads();
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readfirstlane((int)layer[0]);
    const bool crowded = __builtin_amdgcn_readfirstlane((int)layer[1]) != 0;
    const int zmin = pz0 - 1 - 4 * sz, zmax = pz1 - 1 - 4 * sz;  // corner planes that reach the owned ones
    auto deposit_layer = [&](auto* acc, auto crowd) {
      using A = typename std::remove_pointer<decltype(acc)>::type;
      using W = std::conditional_t<NCHI == 1, uint32_t, unsigned long long>;  // weights, and their sum over 64 lanes
      using Word = Codes<NCHI, 1>;  // its first plane is the same for every velocity code
      // lane l takes the particles l len + wave, l len + wave + NW, ... of the layer: the lanes of a
      // wavefront add to different parts of the column (64 neighbours in storage order take 1907 us with
      // 512^3 clustered particles, runs of 16 and 4 lanes 1681 and 1251, this 993), and each lane's cell
      // follows by a cursor that moves forward only
      constexpr uint32_t NW = BLK / 64;
      const uint32_t len = (tot + 63u) / 64u, b0 = (uint32_t)lane * len, e0 = min(b0 + len, tot);
      int cur = 0;
      uint32_t cend = 0;
      {
        const uint32_t i = min(b0 + (uint32_t)wave, tot - 1u);
        int hi = DRC;
        while (hi - cur > 1) {
          const int mid = (cur + hi) >> 1;
          if (cbeg[mid] <= i) cur = mid;
          else hi = mid;
        }
        cend = cbeg[cur + 1];
      }
      // source cell and position word of this lane's particle o (past its last one: some particle)
      auto fetch = [&](uint32_t o, int& sc, Word& w) {
        const uint32_t i = min(b0 + o, tot - 1u);
        while (cend <= i) cend = cbeg[++cur + 1];
        sc = cur;
        w.load_chi(a.codes, (int64_t)(crel[cur] + i));
      };
      auto deposit_one = [&](const bool active, const int s, const Word& w) {
        int ch[3];
        w.chi(ch);
        // corner relative to the source cell (-1 .. 3) and weight numerators
        int i0[3];
        uint32_t w1[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int pl = 2 * ch[d] + 1 - (1 << (SH - 1));
          i0[d] = pl >> SH;
          w1[d] = (uint32_t)pl & ((1u << SH) - 1u);
        }
        const int sx = s % DR, sy = s / DR;
        const int gx = 4 * sx + i0[0] - 3, gy = 4 * sy + i0[1] - 3;  // 0 .. DF: reaches the column
        const bool reach = active && (unsigned)gx <= (unsigned)DF && (unsigned)gy <= (unsigned)DF && i0[2] >= zmin && i0[2] <= zmax;
        int sl = first + 1 + i0[2];
        sl = sl >= NSLOT ? sl - NSLOT : sl;
        const int at = corner[s] + i0[1] * PX + i0[0];  // the corner's word in a bordered plane
        const int up = sl + 1 >= NSLOT ? 0 : sl + 1;
        const uint32_t one = 1u << SH;
        const uint32_t wy2[2] = {one - w1[1], w1[1]}, wx2[2] = {one - w1[0], w1[0]}, wz2[2] = {one - w1[2], w1[2]};
        // weight products: < 2^(3 SH) -- 24-bit factors for 1-byte codes, one 64-bit product else
        auto weight = [&](int j) {
          const uint32_t wzy = NCHI == 1 ? __umul24(wz2[j >> 2], wy2[(j >> 1) & 1]) : wz2[j >> 2] * wy2[(j >> 1) & 1];
          return NCHI == 1 ? (W)__umul24(wzy, wx2[j & 1]) : (W)((unsigned long long)wzy * (unsigned long long)wx2[j & 1]);
        };
        auto word = [&](int j) { return ((j >> 2) ? up : sl) * PLANE + at + ((j >> 1) & 1) * PX + (j & 1); };
        // An LDS add takes 2 cycles per lane on one address. Where MANY lanes or more share a corner cell (the
        // core of a halo: all 64 in the worst case, 1000 cycles for the eight adds) their weights are
        // summed over the wavefront first
        unsigned long long todo = __ballot(reach);
        const int key = sl * PLANE + at;
        const int key_up = up * PLANE + at;
        while (decltype(crowd)::value && todo) {
          // the crowd's two words, from its first lane while every lane is active
          const int first_lane = __ffsll((long long)todo) - 1;
          const int lead = __builtin_amdgcn_readlane(key, first_lane), lead_up = __builtin_amdgcn_readlane(key_up, first_lane);
          const unsigned long long same = __ballot(key == lead) & todo;
          if (__popcll(same) < MANY) break;
          const bool in = (same >> lane) & 1ull;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const W t = wave_total(in ? weight(j) : (W)0);
            if (lane == 63 - j) atomicAdd(acc + ((j >> 2) ? lead_up : lead) + ((j >> 1) & 1) * PX + (j & 1), (A)t);
          }
          todo &= ~same;
        }
        if (decltype(crowd)::value ? (todo >> lane) & 1ull : reach) {
#pragma unroll
          for (int j = 0; j < 8; ++j) atomicAdd(acc + word(j), (A)weight(j));
        }
      };
      // software pipeline, unrolled twice so that the two particles' registers alternate: a wavefront
      // requests the codes of its next chunk before it adds the current one
      uint32_t o = (uint32_t)wave;
      if (o < len) {
        int s0, s1;
        Word w0, w1;
        fetch(o, s0, w0);
        while (true) {
          const uint32_t o1 = o + NW;
          if (o1 < len) fetch(o1, s1, w1);
          deposit_one(b0 + o < e0, s0, w0);
          if (o1 >= len) break;
          o = o1 + NW;
          if (o < len) fetch(o, s0, w0);
          deposit_one(b0 + o1 < e0, s1, w1);
          if (o >= len) break;
        }
      }
    };
    if (tot > 0u) {
      if (narrow && !crowded) deposit_layer(rho32, std::false_type{});
      else if (narrow) deposit_layer(rho32, std::true_type{});
      else if (!crowded) deposit_layer(rho, std::false_type{});
      else deposit_layer(rho, std::true_type{});
    }
    __syncthreads();
    // planes 4 sz - 1 .. 4 sz + 2 are complete: write the owned ones, clear all (what the borders
    // collect is never read)
    static_assert(BLK == DF * DF, "a thread converts one column of fine cells");
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) {
      const int pz = 4 * sz - 1 + pl;
      int sl = first + pl;
      sl = sl >= NSLOT ? sl - NSLOT : sl;
      const int idx = sl * PLANE + mine;
      double r;
      if (narrow) {
        r = (double)rho32[idx];
        rho32[idx] = 0u;
      } else {
        r = (double)rho[idx];
        rho[idx] = 0ull;
      }
      if (pz >= pz0 && pz < pz1) (a.mesh + (int64_t)pz * a.nm * a.pitch_f)[out] = (float)(r * a.inv_mean - 1.0);
    }
    __syncthreads();
  }
}

template <int NCHI, int DTX, int BLK>
__global__ __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(8))) void k_deposit(DepArgs a) {
  deposit_column<NCHI, DTX, BLK>(a, xcd_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y));
}

// every box of an ensemble in one launch (a box's workgroups: its columns times its z chunks)
template <int NCHI, int DTX, int BLK>
__global__ __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(8))) void k_deposit_boxes(BoxTable<DepArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  deposit_column<NCHI, DTX, BLK>(t.args[b], l - t.first[b]);
}

// ---------------------------------------------------------------------------------------------
// Move passes. MODE 0: kick with the potential in the mesh + drift; MODE 1: drift only;
// MODE 2: initial conditions (lattice + Zel'dovich displacement).
// ---------------------------------------------------------------------------------------------
struct MoveArgs {
  const void* codes;
  const uint32_t* cnt;
  const uint64_t* off;
  const float* vc;
  const float* vs;
  void* codes_n;
  const uint64_t* off_n;
  const float* vc_n;
  const float* vinv;
  int64_t cap;
  const float* mesh;
  int64_t pitch_f;
  int nm, nc, nt;
  int64_t nc3;
  float kf, df;
  const float* tdec;
  const float* tedge;  // edge table with -inf / +inf sentinels (M + 1 entries)
  int vhalf;
  uint32_t* mig;  // per (displacement, source cell): counts after the count pass, slots after the link
  int64_t* mom;   // count pass: four moments per cell of a tile and its ring, a block per tile
  uint32_t* flags;
  // initial conditions
  const float* psi0;
  const float* psi1;
  const float* psi2;
  int64_t lat_pitch_f;
  int np, q;
  float vfac, lunit;
  // device-side schedule (replayable step graphs): when kd is set, the kick and drift factors of
  // step j = *kstep are kd[2 j] and kd[2 j + 1] instead of kf and df
  const float* kd;
  const int* kstep;
  // particle IDs (Sec. 2.1): pid_bytes 0 (none), 4 or 8; stored in the order of chi and nu
  const void* pid;
  void* pid_n;
  int pid_bytes;
  // adaptive time steps: when set, the count pass raises amax[0] to the largest |v|^2 after the
  // kick and amax[1] to the largest |t|^2 of the interpolated gradient (FP32 bit patterns)
  uint32_t* amax;
  // moved particles (step and drift passes): when set, the count pass writes every particle's new
  // velocity, codes and displacement at its storage index, and k_place puts them in their new cells
  // (device-side schedule: read from its step word)
  float4* rec;
  // gradient-tile scatter: polls of the LDS turn word after which a chunk stops waiting for its
  // turn and raises the count error (the wait then ends whatever the other wavefronts do)
  uint32_t turn_limit;
};


__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

__global__ void k_clear_u32(uint32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0u;
}

// the ID of the particle at storage index p (steps), or of lattice particle li of tile cell s
// (initial conditions: the lattice index x + N_p (y + N_p z))
template <int MODE>
__device__ __forceinline__ uint64_t particle_id(const MoveArgs& a, const TileGeom& g, int s, int64_t p, uint32_t li) {
  if constexpr (MODE == 2) {
    const int64_t gx = (int64_t)(g.cx0 + s % T) * a.q + li % a.q;
    const int64_t gy = (int64_t)(g.cy0 + (s / T) % T) * a.q + (li / a.q) % a.q;
    const int64_t gz = (int64_t)(g.cz0 + s / (T * T)) * a.q + li / (a.q * a.q);
    return (uint64_t)(gx + a.np * (gy + a.np * gz));
  } else {
    return a.pid_bytes == 8 ? static_cast<const uint64_t*>(a.pid)[p] : static_cast<const uint32_t*>(a.pid)[p];
  }
}

__device__ __forceinline__ void store_id(const MoveArgs& a, uint64_t dst, uint64_t id) {
  if (a.pid_bytes == 8) static_cast<uint64_t*>(a.pid_n)[dst] = id;
  else static_cast<uint32_t*>(a.pid_n)[dst] = (uint32_t)id;
}

// the kick/drift factors of this launch
__device__ __forceinline__ void resolve_factors(MoveArgs& a) {
  if (a.kd) {
    const int j = *a.kstep;
    a.kf = a.kd[2 * j];
    a.df = a.kd[2 * j + 1];
  }
}

// The records of this launch. They are allocated for a call, so a captured launch reads where they lie.
// The address space is named because the compiler cannot tell it of an address read from memory: with flat
// loads k_place takes 174 us for 256^3 particles on as many cells, with global ones 149.
typedef float rec4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) rec4* Records;
typedef __attribute__((address_space(1))) uint32_t* Records2;  // second plane, behind the first
__device__ __forceinline__ Records records(const MoveArgs& a) {
  const uint64_t r = a.kd ? *reinterpret_cast<const uint64_t*>(a.kstep + 2) : reinterpret_cast<uint64_t>(a.rec);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)r), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(r >> 32));
  return (Records)(((uint64_t)hi << 32) | lo);
}

// rint(x s) as int64 for a power of two s and |x s| < 2^51: adding 1.5 * 2^52 rounds x s to the
// nearest integer (ties to even, as rint does) in the low mantissa bits; the difference of the bit
// patterns is that integer. x s is exact, so the fused multiply-add rounds once, as the sum would.
__device__ __forceinline__ long long rint_ll(double x, double s) {
  const double magic = 6755399441055744.0;
  return __double_as_longlong(__builtin_fma(x, s, magic)) - __double_as_longlong(magic);
}

// fixed-point velocity moments of one particle: rint(v_d 2^32) and sum_d rint(v_d^2 2^24). The
// second needs |v| < 2^13.5 for rint_ll; larger speeds (up to the 2^15 overflow limit) take the
// general conversion, decided per wavefront.
__device__ __forceinline__ void velocity_moments(const float* v, long long* q) {
  const bool big = fabsf(v[0]) >= 8192.0f || fabsf(v[1]) >= 8192.0f || fabsf(v[2]) >= 8192.0f;
  q[3] = 0;
  if (__ballot(big) == 0) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double vd = (double)v[d];
      q[d] = rint_ll(vd, 4294967296.0);
      q[3] += rint_ll(vd * vd, 16777216.0);
    }
  } else {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double vd = (double)v[d];
      q[d] = rint_ll(vd, 4294967296.0);
      q[3] += __double2ll_rn(vd * vd * 16777216.0);
    }
  }
}

// Record of a moved particle, written by the count pass and read by k_place: the velocity after
// the kick (FP32, as the encoding takes it), the new position codes and the displacement code
// (z y x digits of k + 1 in base 3). 16 bytes with 1-byte positions; 2-byte ones put the x and y codes
// into a second plane of 4 bytes.
template <int NCHI>
__device__ __forceinline__ void store_record(Records rec, int64_t cap, int64_t p, const float* v, const int* chi, int dcode) {
  const uint32_t w = NCHI == 1 ? (uint32_t)(chi[0] | (chi[1] << 8) | (chi[2] << 16) | (dcode << 24))
                               : (uint32_t)(chi[2] | (dcode << 16));
  rec[p] = rec4{v[0], v[1], v[2], __uint_as_float(w)};
  if constexpr (NCHI == 2) ((Records2)(rec + cap))[p] = (uint32_t)(chi[0] | (chi[1] << 16));
}

struct Moved {
  float v[3];
  int k[3];
  int chi[3];
  bool ok;
};

constexpr int DG = F + 2;  // precomputed-gradient tile side: fine cells -1 .. F of the tile

// Gradient source: either the potential tile (4-point difference per corner) or the tile of
// precomputed unnormalised gradients D = 8 (phi[i+1] - phi[i-1]) - (phi[i+2] - phi[i-2]).
template <bool PRE>
__device__ __forceinline__ float grad_at(const float* ph, const float* gd, int d, int x, int y, int z) {
  // (x, y, z): fine cell relative to the tile origin, in -1 .. F
  if constexpr (PRE) {
    return gd[d * DG * DG * DG + ((z + 1) * DG + (y + 1)) * DG + (x + 1)];
  } else {
    const int e = d == 0 ? 1 : (d == 1 ? PH : PH * PH);
    const int b = ((z + 3) * PH + (y + 3)) * PH + (x + 3);
    const float aa = ph[b + e] - ph[b - e];
    const float bb = ph[b + 2 * e] - ph[b - 2 * e];
    return __builtin_fmaf(8.0f, aa, -bb);  // 8 aa is exact: the same value as 8 aa - bb
  }
}

// New coarse cell along one dimension: k in {-1, 0, 1}, the code of the position inside it, and
// whether the value is usable; a non-finite value, a move beyond one coarse cell or a speed beyond
// the range of the moment accumulators raises its error flag. In range (the usual case) only the
// first branch runs; NaN fails its comparisons.
template <int SH>
__device__ __forceinline__ bool new_cell(float ln, float vd, uint32_t* flags, int& k, int& cq) {
  bool ok = true;
  float lw;
  if (ln >= -4.0f && ln < 8.0f && fabsf(vd) < 32768.0f) {
    k = ln < 0.0f ? -1 : (ln >= 4.0f ? 1 : 0);
    lw = __builtin_fmaf(-4.0f, (float)k, ln);  // ln, ln + 4 or ln - 4, each one rounding
  } else {
    k = 0;
    lw = ln;
    if (!(ln == ln) || fabsf(ln) == INFINITY || !(vd == vd) || fabsf(vd) == INFINITY) {
      set_flag(flags, FLAG_NONFINITE);
      ok = false;
      lw = 0.0f;
    } else if (ln < -4.0f || ln >= 8.0f) {
      set_flag(flags, FLAG_CFL);
      ok = false;
      lw = 0.0f;
    } else if (ln < 0.0f) {
      k = -1;
      lw = ln + 4.0f;
    } else if (ln >= 4.0f) {
      k = 1;
      lw = ln - 4.0f;
    }
    if (fabsf(vd) >= 32768.0f) {
      set_flag(flags, FLAG_OVERFLOW);
      ok = false;
    }
  }
  int q = (int)floorf(lw * (float)(1 << (SH - 1)));
  cq = q < 0 ? 0 : (q > (1 << (SH + 1)) - 1 ? (1 << (SH + 1)) - 1 : q);
  return ok;
}

template <int NCHI, int NNU, int MODE>
__device__ __forceinline__ Moved move_particle(const MoveArgs& a, const float* ph, int s, int64_t p,
                                               uint32_t li, const TileGeom& g) {
  constexpr int SH = 8 * NCHI - 1;
  const int o[3] = {s % T, (s / T) % T, s / (T * T)};
  const int64_t c = (g.cx0 + o[0]) + (int64_t)a.nc * ((g.cy0 + o[1]) + (int64_t)a.nc * (g.cz0 + o[2]));
  float l[3], v[3];
  Moved m;
  if constexpr (MODE == 2) {
    const int lat[3] = {(int)(li % a.q), (int)((li / a.q) % a.q), (int)(li / (a.q * a.q))};
    const int64_t gx = (int64_t)(g.cx0 + o[0]) * a.q + lat[0];
    const int64_t gy = (int64_t)(g.cy0 + o[1]) * a.q + lat[1];
    const int64_t gz = (int64_t)(g.cz0 + o[2]) * a.q + lat[2];
    const int64_t pi = (gz * a.np + gy) * a.lat_pitch_f + gx;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float ps = (d == 0 ? a.psi0 : (d == 1 ? a.psi1 : a.psi2))[pi];
      const float l0 = (float)(2 * lat[d] + 1) * a.lunit;
      v[d] = a.vfac * ps;
      l[d] = l0 + ps;
    }
  } else {
    const float unit = (float)(1.0 / (double)(1 << SH));
    Codes<NCHI, NNU> w;
    w.load(a.codes, a.cap, p);
    int ch[3], nuc[3];
    w.chi(ch);
    w.nu(nuc);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      l[d] = (float)(2 * ch[d] + 1) * unit;
      int nuv = nuc[d];
      nuv = nuv < -a.vhalf ? -a.vhalf : (nuv > a.vhalf ? a.vhalf : nuv);
      v[d] = __builtin_fmaf(a.vs[c], a.tdec[nuv + a.vhalf], a.vc[d * a.nc3 + c]);
    }
    if constexpr (MODE == 0) {
      // CIC corners (fine cells relative to the tile origin) and exact dyadic weights
      int i0[3];
      float w0[3], w1[3];
      const float wunit = (float)(1.0 / (double)(1 << SH));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int pl = o[d] * (1 << (SH + 2)) + 2 * ch[d] + 1 - (1 << (SH - 1));
        i0[d] = pl >> SH;
        const int f = pl & ((1 << SH) - 1);
        w1[d] = (float)f * wunit;
        w0[d] = 1.0f - w1[d];  // exact: both are multiples of 2^-SH in [0, 1]
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        float sacc[2];
#pragma unroll
        for (int cz = 0; cz < 2; ++cz) {
          float racc[2];
#pragma unroll
          for (int cy = 0; cy < 2; ++cy) {
            const float d0 = grad_at<false>(ph, nullptr, d, i0[0], i0[1] + cy, i0[2] + cz);
            const float d1 = grad_at<false>(ph, nullptr, d, i0[0] + 1, i0[1] + cy, i0[2] + cz);
            racc[cy] = __builtin_fmaf(w1[0], d1, w0[0] * d0);
          }
          sacc[cz] = __builtin_fmaf(w1[1], racc[1], w0[1] * racc[0]);
        }
        const float t = __builtin_fmaf(w1[2], sacc[1], w0[2] * sacc[0]);
        v[d] = __builtin_fmaf(t, a.kf, v[d]);
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) l[d] = __builtin_fmaf(v[d], a.df, l[d]);
  }
  m.ok = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    int k, cq;
    if (!new_cell<SH>(l[d], v[d], a.flags, k, cq)) m.ok = false;
    m.k[d] = k;
    m.chi[d] = cq;
    m.v[d] = m.ok ? v[d] : 0.0f;
  }
  return m;
}

// Potential tile (fine cells -3 .. F+2 of the tile, wrapped) and, with PRE, the unnormalised
// 4-point gradient of every corner cell -1 .. F. The gradient uses the same IEEE operations as the
// per-corner evaluation, so both paths give identical bits.
template <int MODE, int NTH>
__device__ __forceinline__ void load_potential(const MoveArgs& a, float* ph, const TileGeom& g) {
  if constexpr (MODE == 0) {
    const int fx0 = g.cx0 * 4 - 3, fy0 = g.cy0 * 4 - 3, fz0 = g.cz0 * 4 - 3;
    const int64_t plane = (int64_t)a.nm * a.pitch_f;
    // all loads of the tile in flight at once, then into LDS
    if (fx0 >= 0 && fy0 >= 0 && fz0 >= 0 && fx0 + PH <= a.nm && fy0 + PH <= a.nm && fz0 + PH <= a.nm &&
        plane < (1 << 26)) {
      // the halo does not cross the box boundary: element e of the tile lies at a 32-bit offset
      // from the tile's first element (below 22 planes of fewer than 2^26 floats); its row index
      // z nm + y and the row pitch are below 2^24, so 24-bit multiplies form the offset
      const float* src = a.mesh + (int64_t)fz0 * plane + (int64_t)fy0 * a.pitch_f + fx0;
      const uint32_t nmu = (uint32_t)a.nm, rs = (uint32_t)a.pitch_f;
      constexpr int NE = PH * PH * PH;
      constexpr int NL = (NE + NTH - 1) / NTH;
      float stage[NL];
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const uint32_t e = threadIdx.x + k * NTH;
        if (NE % NTH == 0 || e < (uint32_t)NE) {
          const uint32_t q = e / PH, x = e - q * PH;
          const uint32_t z = q / PH, y = q - z * PH;
          stage[k] = src[__umul24(__umul24(z, nmu) + y, rs) + x];
        }
      }
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const uint32_t e = threadIdx.x + k * NTH;
        if (NE % NTH == 0 || e < (uint32_t)NE) ph[e] = stage[k];
      }
    } else {
      // half-waves take rows (z, y), wrapped periodically; lanes take x
      const int hw = threadIdx.x >> 5, x = threadIdx.x & 31;
      const int gx = wrapi(fx0 + x, a.nm);
      constexpr int NR = (PH * PH + NTH / 32 - 1) / (NTH / 32);
      float stage[NR];
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int r = hw + k * (NTH / 32);
        if (x < PH && r < PH * PH) {
          const int z = r / PH, y = r - z * PH;
          const int gy = wrapi(fy0 + y, a.nm), gz = wrapi(fz0 + z, a.nm);
          stage[k] = a.mesh[((int64_t)gz * a.nm + gy) * a.pitch_f + gx];
        }
      }
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int r = hw + k * (NTH / 32);
        if (x < PH && r < PH * PH) ph[r * PH + x] = stage[k];
      }
    }
  }
}

// own cells of the tile: counts, starts and the exclusive prefix
template <int MODE>
__device__ __forceinline__ uint32_t own_cells(const MoveArgs& a, const TileGeom& g, uint32_t* pre, uint64_t* start,
                                              uint32_t* wsum) {
  uint32_t cntv = 0;
  if (threadIdx.x < TC) {
    const int s = threadIdx.x;
    const int64_t c = (g.cx0 + s % T) + (int64_t)a.nc * ((g.cy0 + (s / T) % T) + (int64_t)a.nc * (g.cz0 + s / (T * T)));
    if constexpr (MODE == 2) {
      cntv = (uint32_t)(a.q * a.q * a.q);
      start[s] = (uint64_t)c * cntv;
    } else {
      cntv = a.cnt[c];
      start[s] = a.off[c];
    }
  }
  return block_exclusive_scan(cntv, pre, TC, wsum);
}

// Each wave owns a contiguous run of whole cells holding about total/W particles, so that a cell
// is never shared between waves (ranks need no ordering across waves).
__device__ __forceinline__ void wave_cells(const uint32_t* pre, uint32_t total, int wave, int nwaves, int& c0, int& c1) {
  auto lower = [&](uint64_t t) {
    int lo = 0, hi = TC;  // smallest s with pre[s] >= t
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((uint64_t)pre[mid] < t) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  c0 = wave == 0 ? 0 : lower((uint64_t)total * wave / nwaves);
  c1 = wave == nwaves - 1 ? TC : lower((uint64_t)total * (wave + 1) / nwaves);
}

__device__ __forceinline__ int find_cell_in(const uint32_t* pre, int lo, int hi, uint32_t i) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= i) lo = mid;
    else hi = mid;
  }
  return lo;
}


// ---------------------------------------------------------------------------------------------
// Count pass: every particle's kick, drift, new cell and codes, the counts per (source cell,
// displacement) and the fixed-point velocity moments of the new cells. MODE 0: step; 1: drift only;
// 2: initial conditions.
//
// One workgroup per tile of 4^3 coarse cells. The wavefronts take every NW-th chunk of 64 of the
// tile's particles, its cells one after the other in storage order, so that a crowded cell is shared
// by all of them and few particles in a cell leave no lanes idle; nothing here depends on the order.
// The moments of stayers go to CCOPY copies per cell of the LDS accumulators, a lane to copy
// lane % CCOPY: an LDS add takes 2 cycles per lane on one address (128 for a wavefront inside one
// cell), 16 with eight copies, on a pipe beside the vector ALU. Particles that leave their cell add to
// one accumulator per cell of the tile and its ring. A tile writes all its sums to its own block of the
// moment table, and the link adds up the (at most eight) blocks that can reach a cell: no device atomics.
// Stayers are not counted at all (the cell's particles less those that leave).
//
// The potential tile (fine cells -4 .. 19 along x, -3 .. 18 along y and z) is loaded and kept in quads
// of four floats along x, which never straddle the box's edge. Its plane pitch of 540 floats spreads
// the stencils of a cell's particles over the LDS banks (8.0 cycles a read of 64 lanes on average
// over uniform positions; 9.6 with 528).
//
// A tile's loads are in flight together: counts, potential, then, as soon as the counts are there, the
// codes of each wavefront's first chunk, and one barrier for all of it (with the codes requested behind
// that barrier 96^3 on 192^3 39 -> 36 us, 128^3 on 256^3 65 -> 62, 256^3 on 512^3 672 -> 660).
// Two workgroups of 16 wavefronts share a CU (64 VGPRs; workgroups of 8 and 12 take 3 to 12% longer
// where cells hold many particles). Before (512 threads, moments by wavefront prefix scans and device
// atomics) and now: 512^3 particles on 512^3 cells 2291 -> 1647 us early, 2838 -> 1750 clustered, 374 vector
// instructions per 64 particles where there were 535 to 582; 256^3 on 512^3 cells 871 -> 692 us, bound by
// the latencies of the tile's set-up and flush; with step maxima, 96^3 on 128^3, 392 -> 28 us (an atomic
// pair on one address per 64 particles before, one per tile now).
// ---------------------------------------------------------------------------------------------
constexpr int CNTH = kCountThreads;  // threads per workgroup
constexpr int CCOPY = 8;         // copies of an own cell's moment accumulators
constexpr int CPX = F + 8;       // potential row in LDS: 24 floats
constexpr int CPP = PH * CPX + 12;  // potential plane in LDS
constexpr int CSLOT = TC * CCOPY + RC;  // accumulators per moment: own cells' copies, then tile and ring

template <int NCHI, int NNU, int MODE, bool MEAS>
__device__ __forceinline__ void count_tile(MoveArgs a, const unsigned lb) {
  resolve_factors(a);
  const Records rec = MODE != 2 ? records(a) : nullptr;
  constexpr int SH = 8 * NCHI - 1;
  constexpr int NW = CNTH / 64;
  __shared__ __align__(16) float ph[MODE == 0 ? PH * CPP : 4];
  __shared__ __align__(16) unsigned long long mom[4 * CSLOT];
  __shared__ __align__(16) uint32_t left[TC * 27];  // particles leaving own cell s with displacement d (not 13)
  __shared__ float4 cellv[TC];                      // mean velocity and decode scale of the own cells
  __shared__ float tdec_lds[NNU == 1 ? 255 : 1];
  __shared__ uint32_t top[2];
  const bool failed = earlier_phase_failed(a.flags);  // requested first, tested with the counts
  const TileGeom g = tile_of((int)lb, a.nt);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // own cell `lane`, in every wavefront: count and storage start
  // (its index is formed anew where it is used next: kept, it is one register too many)
  auto own_cell = [&] {
    int l = lane, ox, oy, oz;
    asm volatile("" : "+v"(l));
    tile_xyz(l, ox, oy, oz);
    return (uint32_t)(g.cx0 + ox) + (uint32_t)a.nc * ((uint32_t)(g.cy0 + oy) + (uint32_t)a.nc * (uint32_t)(g.cz0 + oz));
  };
  const uint32_t oc = own_cell();
  uint32_t cnt;
  uint64_t beg = 0;  // initial conditions: the lattice particles of a cell are numbered from 0
  if constexpr (MODE == 2) {
    cnt = (uint32_t)(a.q * a.q * a.q);
  } else {
    cnt = a.cnt[oc];
    beg = a.off[oc];
  }
  // Potential: every load of the tile in flight at once, in this order without a branch around them (past
  // the end a load repeats the last row's), so that waiting for the counts does not wait for them. A thread
  // loads the same quad of x in rows 170 apart (7 planes and 16 rows)
  constexpr uint32_t QX = CPX / 4, NR = PH * PH, RPK = CNTH / QX, NL = (NR + RPK - 1) / RPK;
  typedef float quad __attribute__((ext_vector_type(4)));  // (an array of float4 goes to scratch memory here)
  quad stage[MODE == 0 ? NL : 1];
  const uint32_t r0 = min(threadIdx.x / QX, RPK - 1u), qx = threadIdx.x % QX;
  if constexpr (MODE == 0) {
    const uint32_t gx = (uint32_t)wrapi(4 * (g.cx0 - 1) + 4 * (int)qx, a.nm);
    uint32_t z = r0 / PH, y = r0 - z * PH;
#pragma unroll
    for (uint32_t k = 0; k < NL; ++k) {
      if (k) {
        z += RPK / PH;
        y += RPK % PH;
        if (y >= (uint32_t)PH) {
          y -= PH;
          ++z;
        }
        if (k == NL - 1 && z >= (uint32_t)PH) {
          z = PH - 1;
          y = PH - 1;
        }
      }
      const uint32_t gy = (uint32_t)wrapi(4 * g.cy0 - 3 + (int)y, a.nm), gz = (uint32_t)wrapi(4 * g.cz0 - 3 + (int)z, a.nm);
      stage[k] = *reinterpret_cast<const quad*>(a.mesh + ((uint64_t)(__umul24(gz, (uint32_t)a.nm) + gy) * (uint32_t)a.pitch_f + gx));
    }
  }
  for (int i = threadIdx.x; i < 2 * CSLOT; i += CNTH) reinterpret_cast<uint4*>(mom)[i] = make_uint4(0u, 0u, 0u, 0u);
  for (int i = threadIdx.x; i < TC * 27 / 4; i += CNTH) reinterpret_cast<uint4*>(left)[i] = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x < 2) top[threadIdx.x] = 0u;
  if (failed) return;
  if constexpr (MODE != 2) {
    // no code is read and no record written past the end of storage, whatever the counts say
    if (__ballot(beg + cnt > (uint64_t)a.cap)) {
      if (threadIdx.x == 0) set_flag(a.flags, FLAG_COUNT);
      return;
    }
  }
  // inclusive prefix of the counts over the own cells, in the lanes of every wavefront
  const uint32_t inc = (uint32_t)wave_scan_u64(cnt);
  const uint64_t rel = beg - (inc - cnt);  // storage index of a cell's particle i of the tile: rel + i
  const uint32_t rel_lo = (uint32_t)rel, rel_hi = (uint32_t)(rel >> 32);
  const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  const float* const tdec = NNU == 1 ? tdec_lds : a.tdec;
  const float unit = (float)(1.0 / (double)(1 << SH));

  // cell and storage index of each lane's particle of the chunk at c0 (lanes past the end: the tile's
  // last particle)
  auto locate = [&](uint32_t c0, int& sc, int64_t& p) {
    int q = min((int)__popcll(__ballot(inc <= c0)), 63);  // the cell of the chunk's first particle
    uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)inc, q);
    const uint32_t i = min(c0 + (uint32_t)lane, max(tot, 1u) - 1u);
    sc = q;
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)rel_lo, q), hi = (uint32_t)__builtin_amdgcn_readlane((int)rel_hi, q);
    const uint32_t stop = min(c0 + 64u, tot);
    while (end < stop) {
      const uint32_t b = end;  // first particle of the next cell
      ++q;
      end = (uint32_t)__builtin_amdgcn_readlane((int)inc, q);
      const uint32_t ql = (uint32_t)__builtin_amdgcn_readlane((int)rel_lo, q), qh = (uint32_t)__builtin_amdgcn_readlane((int)rel_hi, q);
      if (i >= b) {
        sc = q;
        lo = ql;
        hi = qh;
      }
    }
    p = tot ? (int64_t)((((uint64_t)hi << 32) | lo) + i) : 0;
  };

  float vmax = 0.0f, gmax = 0.0f;  // largest |v|^2 and |t|^2 of this lane's particles
  Codes<NCHI, NNU> wn{0u, 0u, 0u, 0u};
  int sn = 0;
  int64_t pn = 0;
  // the codes of the first chunk are requested before the potential has arrived (wavefronts without a
  // chunk request the codes of the tile's last particle or, of an empty tile, of storage's first)
  uint32_t c0 = 64u * (uint32_t)wave;
  if constexpr (MODE == 2) {
    if (c0 < tot) locate(c0, sn, pn);
  } else {
    locate(min(c0, max(tot, 1u) - 1u), sn, pn);
    wn.load(a.codes, a.cap, pn);
    if (NNU == 1 && threadIdx.x < 255) tdec_lds[threadIdx.x] = a.tdec[threadIdx.x];
    if (threadIdx.x < TC) {
      const uint32_t c = own_cell();
      cellv[threadIdx.x] = make_float4(a.vc[c], (a.vc + a.nc3)[c], (a.vc + 2 * a.nc3)[c], a.vs[c]);
    }
  }
  if constexpr (MODE == 0) {
    if (threadIdx.x < QX * RPK) {
#pragma unroll
      for (uint32_t k = 0; k < NL; ++k) {
        const uint32_t r = r0 + k * RPK;  // plane r / PH by a reciprocal that holds up to NR
        if (k < NL - 1 || r < NR)
          *reinterpret_cast<quad*>(&ph[__umul24(r, CPX) + (CPP - PH * CPX) * (__umul24(r, 65536 / PH + 1) >> 16) + 4u * qx]) = stage[k];
      }
    }
  }
  __syncthreads();
  auto chunk = [&](auto full, uint32_t c0) {
    constexpr bool FULL = decltype(full)::value;
    const int s = sn;
    const int64_t pc = pn;
    int ch[3], nuc[3];
    if constexpr (MODE != 2) {
      wn.chi(ch);
      wn.nu(nuc);
    }
    // the codes of the wavefront's next chunk are requested before this one's record is stored (past
    // the end the request repeats a particle of this chunk)
    if (c0 + 64u * NW < tot) locate(c0 + 64u * NW, sn, pn);
    if constexpr (MODE != 2) wn.load(a.codes, a.cap, pn);
    const bool active = FULL || c0 + (uint32_t)lane < tot;
    int o[3];
    tile_xyz(s, o[0], o[1], o[2]);
    float v[3], l[3];
    if constexpr (MODE == 2) {
      const uint32_t li = (uint32_t)pc, q = (uint32_t)a.q;
      const int lat[3] = {(int)(li % q), (int)((li / q) % q), (int)(li / (q * q))};
      const int64_t pi = ((int64_t)((g.cz0 + o[2]) * a.q + lat[2]) * a.np + ((g.cy0 + o[1]) * a.q + lat[1])) * a.lat_pitch_f +
                         ((g.cx0 + o[0]) * a.q + lat[0]);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const float ps = (d == 0 ? a.psi0 : (d == 1 ? a.psi1 : a.psi2))[pi];
        v[d] = a.vfac * ps;
        l[d] = (float)(2 * lat[d] + 1) * a.lunit + ps;
      }
    } else {
      const float4 cv = cellv[s];
      const float vcv[3] = {cv.x, cv.y, cv.z};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        int nuv = nuc[d];
        nuv = nuv < -a.vhalf ? -a.vhalf : (nuv > a.vhalf ? a.vhalf : nuv);
        l[d] = (float)(2 * ch[d] + 1) * unit;
        v[d] = __builtin_fmaf(cv.w, tdec[nuv + a.vhalf], vcv[d]);
      }
    }
    float vv = 0.f, tq = 0.f;
    if constexpr (MODE == 0) {
      // CIC corner relative to the tile, exact dyadic weights, interpolated gradient
      int i0[3];
      float w0[3], w1[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int pl = o[d] * (1 << (SH + 2)) + 2 * ch[d] + 1 - (1 << (SH - 1));
        i0[d] = pl >> SH;
        w1[d] = (float)(pl & ((1 << SH) - 1)) * unit;
        w0[d] = 1.0f - w1[d];  // exact: both are multiples of 2^-SH in [0, 1]
      }
      const float* const corner = &ph[(i0[2] + 3) * CPP + (i0[1] + 3) * CPX + (i0[0] + 4)];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        constexpr int st[3] = {1, CPX, CPP};
        const int e = st[d];
        auto grad = [&](int x, int y, int z) {
          const float* const f = corner + x + CPX * y + CPP * z;
          const float aa = f[e] - f[-e], bb = f[2 * e] - f[-2 * e];
          return __builtin_fmaf(8.0f, aa, -bb);  // 8 aa is exact: the same value as 8 aa - bb
        };
        float sacc[2];
#pragma unroll
        for (int cz = 0; cz < 2; ++cz) {
          float racc[2];
#pragma unroll
          for (int cy = 0; cy < 2; ++cy) racc[cy] = __builtin_fmaf(w1[0], grad(1, cy, cz), w0[0] * grad(0, cy, cz));
          sacc[cz] = __builtin_fmaf(w1[1], racc[1], w0[1] * racc[0]);
        }
        const float t = __builtin_fmaf(w1[2], sacc[1], w0[2] * sacc[0]);
        v[d] = __builtin_fmaf(t, a.kf, v[d]);
        if constexpr (MEAS) tq = d == 0 ? t * t : tq + t * t;
      }
      if constexpr (MEAS) vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    }
    if constexpr (MEAS) {
      vmax = fmaxf(vmax, active ? vv : 0.0f);
      gmax = fmaxf(gmax, active ? tq : 0.0f);
    }
    if constexpr (MODE != 2) {
#pragma unroll
      for (int d = 0; d < 3; ++d) l[d] = __builtin_fmaf(v[d], a.df, l[d]);
    }
    // New cell and codes; the fast way when every particle of the chunk moves by at most one cell at a
    // speed that both moment roundings take (NaN fails the comparisons)
    int k[3], cq[3];
    long long q[4];
    bool usual = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) usual = usual & (l[d] >= -4.0f) & (l[d] < 8.0f) & (fabsf(v[d]) < 8192.0f);
    if (__ballot(!usual) == 0ull) {
      q[3] = 0;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const float kf = floorf(0.25f * l[d]);  // -1, 0 or 1
        const int c = (int)floorf(__builtin_fmaf(-4.0f, kf, l[d]) * (float)(1 << (SH - 1)));
        k[d] = (int)kf;
        cq[d] = min(max(c, 0), (1 << (SH + 1)) - 1);
        const double vd = (double)v[d];
        q[d] = rint_ll(vd, 4294967296.0);
        q[3] += rint_ll(vd * vd, 16777216.0);
      }
    } else {
      bool ok = true;
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (!new_cell<SH>(active ? l[d] : 0.0f, active ? v[d] : 0.0f, a.flags, k[d], cq[d])) ok = false;
#pragma unroll
      for (int d = 0; d < 3; ++d) v[d] = ok ? v[d] : 0.0f;
      velocity_moments(v, q);
    }
    const int dcode = 13 + k[0] + 3 * k[1] + 9 * k[2];
    const bool stay = dcode == 13;
    const int ring = 43 + o[0] + RG * o[1] + RG * RG * o[2] + k[0] + RG * k[1] + RG * RG * k[2];
    const int slot = stay ? s * CCOPY + (lane & (CCOPY - 1)) : TC * CCOPY + ring;
    if (active) {
      if constexpr (MODE != 2)
        if (rec) store_record<NCHI>(rec, a.cap, pc, v, cq, dcode);
#pragma unroll
      for (int d = 0; d < 4; ++d) atomicAdd(&mom[d * CSLOT + slot], (unsigned long long)q[d]);
      if (!stay) atomicAdd(&left[s * 27 + dcode], 1u);
    }
  };
  for (; c0 + 64u <= tot; c0 += 64u * NW) chunk(std::true_type{}, c0);
  if (c0 < tot) chunk(std::false_type{}, c0);
  if constexpr (MEAS) {
    // one pair of device atomics per tile, and none once the maxima are higher
    vmax = wave_max(vmax);
    gmax = wave_max(gmax);
    if (lane == 0) {
      atomicMax(&top[0], __float_as_uint(vmax));
      atomicMax(&top[1], __float_as_uint(gmax));
    }
  }
  __syncthreads();
  if constexpr (MEAS) {
    if (threadIdx.x < 2 && top[threadIdx.x] > __atomic_load_n(&a.amax[threadIdx.x], __ATOMIC_RELAXED))
      atomicMax(&a.amax[threadIdx.x], top[threadIdx.x]);
  }
  // moments of the tile's and the ring's new cells, four to a cell
  unsigned long long* const out = reinterpret_cast<unsigned long long*>(a.mom) + (uint64_t)lb * (4 * RC);
  for (int i = threadIdx.x; i < 4 * RC; i += CNTH) {
    const int d = i & 3, r = i >> 2;
    const int rx = r % RG - 1, ry = (r / RG) % RG - 1, rz = r / (RG * RG) - 1;
    unsigned long long v = mom[d * CSLOT + TC * CCOPY + r];
    if ((unsigned)rx < (unsigned)T && (unsigned)ry < (unsigned)T && (unsigned)rz < (unsigned)T) {
      const ulonglong2* const m = reinterpret_cast<const ulonglong2*>(&mom[d * CSLOT + (rx + T * (ry + T * rz)) * CCOPY]);
#pragma unroll
      for (int j = 0; j < CCOPY / 2; ++j) v += m[j].x + m[j].y;
    }
    out[i] = v;
  }
  // counts: a wavefront writes one displacement of all own cells, a lane per cell; the wavefront that
  // has displacement 13 takes the leavers from the cell's count
  uint32_t* const col = a.mig + own_cell();
  for (int d = wave; d < 27; d += NW) {
    uint32_t n = left[lane * 27 + d];
    if (d == 13) {
      const uint32_t below = (uint32_t)__shfl_up((int)inc, 1);
      n = inc - (lane ? below : 0u);  // the cell's count
      for (int j = 0; j < 27; ++j) n -= left[lane * 27 + j];  // entry 13 stays 0
    }
    (col + d * a.nc3)[0] = n;
  }
}

template <int NCHI, int NNU, int MODE, bool MEAS = false>
__global__ __launch_bounds__(CNTH) __attribute__((amdgpu_waves_per_eu(8))) void k_count(MoveArgs a) {
  count_tile<NCHI, NNU, MODE, MEAS>(a, xcd_block(blockIdx.x, gridDim.x));
}

// every box of an ensemble in one launch (a box's workgroups: its tiles)
template <int NCHI, int NNU>
__global__ __launch_bounds__(CNTH) __attribute__((amdgpu_waves_per_eu(8))) void k_count_boxes(BoxTable<MoveArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  count_tile<NCHI, NNU, 0, false>(t.args[b], l - t.first[b]);
}

// Eq. (nu): the codes nu with ext[nu + h] <= u < ext[nu + h + 1] (h = (M-1)/2; ext is the edge table with
// -inf and +inf at its ends). x = (M / pi) atan(u) in FP32 (atan z = z P(z^2) on [0, 1], eight
// coefficients of a near-minimax fit: its error alternates over nine extrema of 2.7e-8 to 4.8e-8;
// M / 2 - x(1 / u) beyond) is off by at most 2e-5 codes for M = 255 and 0.005
// for M = 65535 (over every edge, its neighbours and 2e7 other floats, the reciprocal up to an ulp off). So
// the nearest integer is the code unless x lies close to the middle of two, where the table decides:
// 0.02 and 2.4 in a hundred. Against a bucket table, whose entry two exact steps then corrected (five
// reads a code in a chain of three, of 768 KB of tables for M = 65535), k_place takes, in us: 2-byte codes
// and IDs, 96^3 on 192^3, 46 -> 21 (clustered 72 -> 38); 1-byte codes 128^3 on 256^3 34 -> 32, 256^3 on 256^3
// clustered 239 -> 227.
template <int NNU>
__device__ __forceinline__ void encode_nu3(const float* u, const float* ext, int vhalf, int* nu) {
  constexpr float M = NNU == 1 ? 255.0f : 65535.0f, H = 0.5f * (M - 1.0f);
  constexpr double mp = (NNU == 1 ? 255.0 : 65535.0) / 3.14159265358979323846;
  constexpr float sure = 0.5f - (NNU == 1 ? 1e-4f : 0.012f);
  constexpr float c[8] = {(float)(0.9999993443489075 * mp),   (float)(-0.33329859375953674 * mp),
                          (float)(0.19946563243865967 * mp),  (float)(-0.13908620178699493 * mp),
                          (float)(0.09642171859741211 * mp),  (float)(-0.05591198801994324 * mp),
                          (float)(0.021862726658582687 * mp), (float)(-0.004054504446685314 * mp)};
  bool near = false;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float a = fabsf(u[d]);
    const float z = fminf(a, __builtin_amdgcn_rcpf(a)), w = z * z;
    float p = c[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) p = __builtin_fmaf(p, w, c[k]);
    const float zp = z * p;
    const float x = copysignf(a > 1.0f ? 0.5f * M - zp : zp, u[d]);
    const float r = rintf(x);
    near = near | !(fabsf(x - r) <= sure);
    nu[d] = (int)fminf(fmaxf(r, -H), H);  // (NaN: -h)
  }
  if (near) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float* const e = ext + (nu[d] + vhalf);
      nu[d] = min(nu[d] + (int)(u[d] >= e[1]) - (int)(u[d] < e[0]), vhalf);
    }
  }
}

template <int NCHI, int NNU, int MODE, int NTH>
__device__ __forceinline__ void move_scatter_tile(MoveArgs a, const unsigned lb) {
  resolve_factors(a);
  __shared__ float ph[MODE == 0 ? PH * PH * PH : 1];
  __shared__ uint32_t grp[TC * 27];
  __shared__ uint32_t pre[TC + 1];
  __shared__ uint64_t start[TC];
  __shared__ uint32_t wsum[NTH / 64];
  __shared__ float edges_lds[NNU == 1 ? 256 : 1];
  // the flag word is requested first and tested after the set-up (the last barrier): a wave that
  // returns then cannot hold up the others
  const uint32_t failed = __atomic_load_n(a.flags, __ATOMIC_RELAXED);
  const TileGeom g = tile_of(lb, a.nt);
  load_potential<MODE, NTH>(a, ph, g);
  for (int i = threadIdx.x; i < TC * 27; i += NTH) grp[i] = 0u;
  const int nedge = 2 * a.vhalf + 2;
  if constexpr (NNU == 1)
    for (int i = threadIdx.x; i < nedge; i += NTH) edges_lds[i] = a.tedge[i];
  const float* edges = (NNU == 1) ? edges_lds : a.tedge;
  const uint32_t total = own_cells<MODE>(a, g, pre, start, wsum);
  if (__builtin_amdgcn_readfirstlane(failed)) return;  // a failed step is not applied
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long lt = (1ull << lane) - 1ull;
  int c0, c1;
  wave_cells(pre, total, wave, NTH / 64, c0, c1);
  const uint32_t p0 = pre[c0], p1 = pre[c1];
  // particles of this wave's cells in storage order; the running count per (source cell,
  // displacement) gives every particle its rank inside the new cell
  for (uint32_t base = p0; base < p1; base += 64) {
    const uint32_t i = base + lane;
    const bool active = i < p1;
    Moved m{};
    int s = c0, key = 0, dcode = 0;
    if (active) {
      s = find_cell_in(pre, c0, c1, i);
      const uint32_t li = i - pre[s];
      const int64_t p = (int64_t)start[s] + li;
      m = move_particle<NCHI, NNU, MODE>(a, ph, s, p, li, g);
      dcode = (m.k[2] + 1) * 9 + (m.k[1] + 1) * 3 + (m.k[0] + 1);
      key = s * 27 + dcode;
    }
    unsigned long long peers = __ballot(active);
#pragma unroll
    for (int b = 0; b < 11; ++b) {
      const bool bit = (key >> b) & 1;
      const unsigned long long bb = __ballot(active && bit);
      peers &= bit ? bb : ~bb;
    }
    const int rin = __popcll(peers & lt);
    const int leader = active ? __ffsll((long long)peers) - 1 : lane;
    uint32_t gbase = 0;
    if (active && rin == 0) {
      gbase = grp[key];
      grp[key] = gbase + (uint32_t)__popcll(peers);
    }
    gbase = (uint32_t)__shfl((int)gbase, leader, 64);
    if (active) {
      int ox, oy, oz;
      tile_xyz(s, ox, oy, oz);
      const int nx = wrapi(g.cx0 + ox + m.k[0], a.nc), ny = wrapi(g.cy0 + oy + m.k[1], a.nc);
      const int nz = wrapi(g.cz0 + oz + m.k[2], a.nc);
      const int64_t cn = nx + (int64_t)a.nc * (ny + (int64_t)a.nc * nz);
      const int64_t co = (g.cx0 + ox) + (int64_t)a.nc * ((g.cy0 + oy) + (int64_t)a.nc * (g.cz0 + oz));
      const uint64_t dst = a.off_n[cn] + a.mig[(int64_t)dcode * a.nc3 + co] + gbase + (uint32_t)rin;
      if (dst < (uint64_t)a.cap) {
        const float inv = a.vinv[cn];
        float u[3];
        int nu[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) u[d] = (m.v[d] - a.vc_n[d * a.nc3 + cn]) * inv;
        encode_nu3<NNU>(u, edges, a.vhalf, nu);
        Codes<NCHI, NNU> w;
        w.set(m.chi, nu);
        w.store(a.codes_n, a.cap, (int64_t)dst);
        if (a.pid_bytes) store_id(a, dst, particle_id<MODE>(a, g, s, (int64_t)start[s] + (i - pre[s]), i - pre[s]));
      } else {
        set_flag(a.flags, FLAG_COUNT);
      }
    }
  }
}

template <int NCHI, int NNU, int MODE, int NTH>
__global__ __launch_bounds__(NTH) void k_move_scatter(MoveArgs a) {
  move_scatter_tile<NCHI, NNU, MODE, NTH>(a, xcd_block(blockIdx.x, gridDim.x));
}

template <int NCHI, int NNU, int MODE, int NTH>
__global__ __launch_bounds__(NTH) void k_move_scatter_boxes(BoxTable<MoveArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  move_scatter_tile<NCHI, NNU, MODE, NTH>(t.args[b], l - t.first[b]);
}

// ---------------------------------------------------------------------------------------------
// Recomputing scatter with the gradient tile (steps without records, where cells hold many particles):
// the 4-point gradient of the whole tile is formed once in LDS, the tile's particles are shared by
// all wavefronts in chunks of 64, and their ranks are taken in storage order.
// ---------------------------------------------------------------------------------------------

template <int NCHI, int NNU>
__device__ __forceinline__ void scatter_dense_tile(MoveArgs a, const unsigned lb) {
  resolve_factors(a);
  constexpr int NTH = 1024;
  constexpr int SH = 8 * NCHI - 1;
  // one region holds the potential tile, then the gradient tile computed from it, so that two
  // workgroups fit a CU
  constexpr int NG = 3 * DG * DG * DG;
  static_assert(PH * PH * PH <= NG, "the potential tile must fit the gradient region");
  __shared__ float tile[NG];
  float* const ph = tile;
  float* const gd = tile;
  __shared__ uint32_t grp[TC * 27];              // particles ranked so far per (cell, displacement)
  __shared__ uint32_t pre[TC + 1];
  __shared__ uint64_t start[TC];
  __shared__ uint32_t wsum[NTH / 64];
  __shared__ float tdec_lds[NNU == 1 ? 255 : 1];
  __shared__ float edges_lds[NNU == 1 ? 256 : 1];
  const TileGeom g = tile_of(lb, a.nt);
  // the flag word is requested first and tested after the set-up (the last barrier)
  const uint32_t failed = __atomic_load_n(a.flags, __ATOMIC_RELAXED);
  // mean velocity and decode scale of the tile's cells
  __shared__ float4 cellv[TC];
  uint32_t cnt_r = 0;  // particle count of own cell threadIdx.x
  {
    // every global read of the set-up in flight at once: the code tables, the own cells' counts,
    // starts, mean velocities and decode scales, then the potential tile
    static_assert(NTH >= 1024 && NTH >= TC, "one table entry and at most one own cell per thread");
    float tdec_r = 0.0f, edge_r = 0.0f;
    if constexpr (NNU == 1) {
      if (threadIdx.x < 255) tdec_r = a.tdec[threadIdx.x];
      if (threadIdx.x < 256) edge_r = a.tedge[threadIdx.x];
    }
    float4 cv_r = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    uint64_t start_r = 0;
    if (threadIdx.x < TC) {
      const int sx = threadIdx.x;
      const int64_t c = (g.cx0 + sx % T) + (int64_t)a.nc * ((g.cy0 + (sx / T) % T) + (int64_t)a.nc * (g.cz0 + sx / (T * T)));
      cnt_r = a.cnt[c];
      start_r = a.off[c];
      cv_r = make_float4(a.vc[c], a.vc[a.nc3 + c], a.vc[2 * a.nc3 + c], a.vs[c]);
    }
    load_potential<0, NTH>(a, ph, g);
    if constexpr (NNU == 1) {
      if (threadIdx.x < 255) tdec_lds[threadIdx.x] = tdec_r;
      if (threadIdx.x < 256) edges_lds[threadIdx.x] = edge_r;
    }
    if (threadIdx.x < TC) {
      cellv[threadIdx.x] = cv_r;
      start[threadIdx.x] = start_r;
    }
  }
  __syncthreads();
  {
    // gradient of every corner cell -1 .. F of the tile, over the potential: the z component lies
    // beyond the potential tile and is stored at once; x and y go through registers
    constexpr int G3 = DG * DG * DG;
    static_assert(2 * G3 >= PH * PH * PH, "the z gradient must not overlap the potential tile");
    constexpr int K = (G3 + NTH - 1) / NTH;
    auto grad_of = [&](int d, int i) {
      const int z = i / (DG * DG), y = (i / DG) % DG, x = i % DG;
      return grad_at<false>(ph, nullptr, d, x - 1, y - 1, z - 1);
    };
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = threadIdx.x + k * NTH;
      if (G3 % NTH == 0 || i < G3) gd[2 * G3 + i] = grad_of(2, i);
    }
    float gx[K], gy[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = threadIdx.x + k * NTH;
      if (G3 % NTH == 0 || i < G3) {
        gx[k] = grad_of(0, i);
        gy[k] = grad_of(1, i);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = threadIdx.x + k * NTH;
      if (G3 % NTH == 0 || i < G3) {
        gd[i] = gx[k];
        gd[G3 + i] = gy[k];
      }
    }
  }
  for (int i = threadIdx.x; i < TC * 27; i += NTH) grp[i] = 0u;
  // [0] the number of the tile's chunks ranked so far, [1] set if a wait gave up
  __shared__ uint32_t turn[2];
  if (threadIdx.x == 0) turn[0] = turn[1] = 0u;
  const float* tdec = NNU == 1 ? tdec_lds : a.tdec;
  const float* edges = NNU == 1 ? edges_lds : a.tedge;
  block_exclusive_scan(cnt_r, pre, TC, wsum);  // ends with a barrier
  if (__builtin_amdgcn_readfirstlane(failed)) return;  // a failed step is not applied
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float unit = (float)(1.0 / (double)(1 << SH));
  // kick, drift, new cell and code of one particle (cell s at tile offsets (ci, o1, o2), codes chc,
  // nuc); inactive lanes keep v = l = 0
  auto physics = [&](bool active, int s, int ci, int o1, int o2, const int* chc, const int* nuc, float* v, int* k,
                     int* cq) {
    float l[3] = {0.f, 0.f, 0.f};
    v[0] = v[1] = v[2] = 0.f;
    int ch[3] = {0, 0, 0};
    if (active) {
      const float4 cv = cellv[s];
      const float vcv[3] = {cv.x, cv.y, cv.z};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        ch[d] = chc[d];
        int nuv = nuc[d];
        nuv = nuv < -a.vhalf ? -a.vhalf : (nuv > a.vhalf ? a.vhalf : nuv);
        l[d] = (float)(2 * ch[d] + 1) * unit;
        v[d] = __builtin_fmaf(cv.w, tdec[nuv + a.vhalf], vcv[d]);
      }
      // CIC corners relative to the tile, exact dyadic weights, interpolated gradient
      const int o[3] = {ci, o1, o2};
      int i0[3];
      float w0[3], w1[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int pl = o[d] * (1 << (SH + 2)) + 2 * ch[d] + 1 - (1 << (SH - 1));
        i0[d] = pl >> SH;
        const int f = pl & ((1 << SH) - 1);
        w1[d] = (float)f * unit;
        w0[d] = 1.0f - w1[d];  // exact: both are multiples of 2^-SH in [0, 1]
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        float sacc[2];
#pragma unroll
        for (int cz = 0; cz < 2; ++cz) {
          float racc[2];
#pragma unroll
          for (int cy = 0; cy < 2; ++cy) {
            const float d0 = grad_at<true>(ph, gd, d, i0[0], i0[1] + cy, i0[2] + cz);
            const float d1 = grad_at<true>(ph, gd, d, i0[0] + 1, i0[1] + cy, i0[2] + cz);
            racc[cy] = __builtin_fmaf(w1[0], d1, w0[0] * d0);
          }
          sacc[cz] = __builtin_fmaf(w1[1], racc[1], w0[1] * racc[0]);
        }
        const float t = __builtin_fmaf(w1[2], sacc[1], w0[2] * sacc[0]);
        v[d] = __builtin_fmaf(t, a.kf, v[d]);
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) l[d] = __builtin_fmaf(v[d], a.df, l[d]);
    }
    // new cell, codes, flags (same rules as the generic path)
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (!new_cell<SH>(l[d], v[d], a.flags, k[d], cq[d])) ok = false;
    if (!ok) {
#pragma unroll
      for (int d = 0; d < 3; ++d) v[d] = 0.0f;
    }
  };
  // The wavefronts take every NW-th chunk of 64 of the tile's particles (its 64 cells
  // in storage order, one after the other), so that a crowded cell is shared by all of them; the
  // lanes of a chunk find their cells from the prefix counts by a forward walk shared by the
  // wavefront.
  {
    constexpr int NW = NTH / 64;
    const uint32_t tot = pre[TC];
    int ec = 0;  // the cell of the chunk's first particle (wave-uniform, non-decreasing)
    auto locate = [&](uint32_t c0, int& sc, int64_t& p) {
      while ((uint32_t)__builtin_amdgcn_readfirstlane(pre[ec + 1]) <= c0) ++ec;
      const uint32_t i = c0 + (uint32_t)lane;
      sc = ec;
      for (int q = ec + 1; q < TC; ++q) {
        const uint32_t pq = (uint32_t)__builtin_amdgcn_readfirstlane(pre[q]);
        if (pq >= c0 + 64u) break;
        if (pq <= i) sc = q;
      }
      // lanes past the end read the chunk's first particle
      p = i < tot ? (int64_t)start[sc] + (i - pre[sc]) : (int64_t)start[ec] + (c0 - pre[ec]);
    };
    Codes<NCHI, NNU> wn{0u, 0u, 0u, 0u};
    auto load_at = [&](int64_t p) { wn.load(a.codes, a.cap, p); };
    uint32_t c0 = 64u * (uint32_t)wave;
    int sn = 0;
    int64_t pn = 0;
    if (c0 < tot) {
      locate(c0, sn, pn);
      load_at(pn);
    }
    for (; c0 < tot; c0 += 64u * NW) {
      const uint32_t i = c0 + (uint32_t)lane;
      const bool active = i < tot;
      const int s = sn;
      const int64_t pc = pn;
      int chc[3], nuc[3];
      wn.chi(chc);
      wn.nu(nuc);
      // the codes of the next chunk are requested before this chunk's atomics and stores are issued
      // (past the end the request repeats a particle of this chunk)
      if (c0 + 64u * NW < tot) locate(c0 + 64u * NW, sn, pn);
      load_at(pn);
      int ci, o1, o2;
      tile_xyz(s, ci, o1, o2);
      float v[3];
      int k[3], cq[3];
      physics(active, s, ci, o1, o2, chc, nuc, v, k, cq);
      const int dcode = (k[2] + 1) * 9 + (k[1] + 1) * 3 + (k[0] + 1);
      {
        // Scatter: the rank inside the (new cell, source offset) slot is the number of the
        // particles before this one in storage order with the same (source cell, displacement).
        // Within the chunk it comes from the lanes with the same key: the cell's lanes are one
        // contiguous range, the displacement is matched with one ballot per bit of its code.
        // Across chunks it comes from the running count per key in LDS, which the chunks update
        // strictly in storage order: chunk c waits until c chunks have been ranked (wavefronts of
        // one workgroup are all resident, and chunk c - 1's wavefront never waits for chunk c, so
        // the wait ends; it is also bounded, and one that gives up raises an error flag).
        const int key = s * 27 + dcode;
        const uint32_t cbeg = pre[s], cend = pre[s + 1];
        const int la = cbeg > c0 ? (int)(cbeg - c0) : 0;  // the cell's lanes: [la, cend - c0)
        const uint32_t le = cend - c0;
        unsigned long long peers =
            __ballot(active) & (le >= 64u ? ~0ull : ((1ull << le) - 1ull)) & ~((1ull << la) - 1ull);
#pragma unroll
        for (int bt = 0; bt < 5; ++bt) {
          const bool bit = (dcode >> bt) & 1;
          const unsigned long long bb = __ballot(active && bit);
          peers &= bit ? bb : ~bb;
        }
        const uint32_t rin = lanes_below(peers), npeer = (uint32_t)__popcll(peers);
        // the lowest lane of the key: it alone advances the key's running count
        const int leader = peers ? __ffsll((long long)peers) - 1 : lane;
        // the ranks are formed before the turn is awaited (the compiler would otherwise move them
        // into the ordered section, which the chunks pass through one at a time)
        asm volatile("" ::"v"(rin), "v"(npeer), "v"(leader));
        // destination cell data, requested before the turn is awaited
        const int nx = wrapi(g.cx0 + ci + k[0], a.nc), ny = wrapi(g.cy0 + o1 + k[1], a.nc);
        const int nz = wrapi(g.cz0 + o2 + k[2], a.nc);
        const int64_t cn = nx + (int64_t)a.nc * (ny + (int64_t)a.nc * nz);
        uint64_t dbase = 0;
        float inv = 0.0f, vcn[3] = {0.0f, 0.0f, 0.0f};
        if (active) {
          const int64_t co = (g.cx0 + ci) + (int64_t)a.nc * ((g.cy0 + o1) + (int64_t)a.nc * (g.cz0 + o2));
          dbase = a.off_n[cn] + a.mig[(int64_t)dcode * a.nc3 + co];
          inv = a.vinv[cn];
#pragma unroll
          for (int d = 0; d < 3; ++d) vcn[d] = a.vc_n[d * a.nc3 + cn];
        }
        const uint32_t chunk = c0 / 64u;
        {
          uint32_t spins = 0;
          while (__hip_atomic_load(&turn[0], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != chunk &&
                 __hip_atomic_load(&turn[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u) {
            __builtin_amdgcn_s_sleep(0);
            if (++spins >= a.turn_limit) {
              if (lane == 0) {
                __hip_atomic_store(&turn[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                set_flag(a.flags, FLAG_COUNT);
              }
              break;
            }
          }
        }
        // the ordered section: one LDS read-modify-write per key (by its lowest lane), then the turn
        // passes on; the key's other lanes take the count from that lane afterwards
        uint32_t b0 = 0u;
        if (active && rin == 0u) b0 = atomicAdd(&grp[key], npeer);
        if (lane == 0) __hip_atomic_store(&turn[0], chunk + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        b0 = (uint32_t)__shfl((int)b0, leader);
        if (active) {
          const uint64_t dst = dbase + b0 + rin;
          if (dst < (uint64_t)a.cap) {
            float u[3];
            int nu[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) u[d] = (v[d] - vcn[d]) * inv;
            encode_nu3<NNU>(u, edges, a.vhalf, nu);
            Codes<NCHI, NNU> w;
            w.set(cq, nu);
            w.store(a.codes_n, a.cap, (int64_t)dst);
            if (a.pid_bytes) store_id(a, dst, particle_id<0>(a, g, s, pc, 0u));
          } else {
            set_flag(a.flags, FLAG_COUNT);
          }
        }
      }
    }
  }
}

// two 1024-thread workgroups per CU: at most 64 VGPRs
template <int NCHI, int NNU>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_scatter_dense(MoveArgs a) {
  scatter_dense_tile<NCHI, NNU>(a, xcd_block(blockIdx.x, gridDim.x));
}

template <int NCHI, int NNU>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_scatter_dense_boxes(BoxTable<MoveArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  scatter_dense_tile<NCHI, NNU>(t.args[b], l - t.first[b]);
}

// ---------------------------------------------------------------------------------------------
// Place: the scatter pass from the count pass's records. A workgroup of four wavefronts takes a tile
// of 4^3 coarse cells, each wavefront one z layer of 16 cells in storage order, 64 particles at a
// time, so the running destination per (source cell, displacement) in LDS is advanced by one
// wavefront only and needs no ordering between wavefronts: the order is that of the recomputing
// passes. Against recomputing the move, the potential tile (42 to 83 bytes per particle where cells
// hold few), the interpolation and the kick are gone for 16 bytes per particle written and read:
// 256^3 particles on 512^3 cells 850 -> 338 us, 512^3 on 512^3 2253 -> 1340 us, for 60 and 110 us
// more in the count pass; 292 and 990 us with the packed codes. Workgroups of 512 and 1024 threads,
// and half as many of them on a CU, take the same time: it is bound by the requests of its stores
// (one per destination line) and by its 185 vector instructions a chunk of 64 particles.
// ---------------------------------------------------------------------------------------------
constexpr int PLACE_BLK = 256;

template <int NCHI, int NNU, bool PID>
__device__ __forceinline__ void place_tile(const MoveArgs& a, const unsigned lb) {
  constexpr int WC = TC / (PLACE_BLK / 64);  // cells per wavefront
  __shared__ uint32_t next[TC * 27];  // next destination per (own cell, displacement)
  __shared__ uint32_t offr[RC];       // of the tile's and ring's new cells: offset,
  __shared__ float4 stat[RC];         // mean velocity and encode scale
  __shared__ float edges_lds[NNU == 1 ? 256 : 1];
  const uint32_t failed = __atomic_load_n(a.flags, __ATOMIC_RELAXED);
  const Records rec = records(a);
  const TileGeom g = tile_of(lb, a.nt);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nc = (uint32_t)a.nc;
  if (threadIdx.x < RC) {
    const int r = threadIdx.x;
    const uint32_t nx = (uint32_t)wrapi(g.cx0 + r % RG - 1, a.nc), ny = (uint32_t)wrapi(g.cy0 + (r / RG) % RG - 1, a.nc);
    const uint32_t nz = (uint32_t)wrapi(g.cz0 + r / (RG * RG) - 1, a.nc);
    const uint32_t c = nx + nc * (ny + nc * nz);
    offr[r] = (uint32_t)a.off_n[c];  // below 2^31 (the records' limit on the capacity)
    stat[r] = make_float4(a.vc_n[c], (a.vc_n + a.nc3)[c], (a.vc_n + 2 * a.nc3)[c], a.vinv[c]);
  }
  // every slot of the tile requested at once: wavefront w takes the displacements w, w + 4, ...
  constexpr int NS = (27 + PLACE_BLK / 64 - 1) / (PLACE_BLK / 64);
  uint32_t sl[NS];
  int ox, oy, oz;
  tile_xyz(lane, ox, oy, oz);
  {
    const uint32_t c = (uint32_t)(g.cx0 + ox) + nc * ((uint32_t)(g.cy0 + oy) + nc * (uint32_t)(g.cz0 + oz));
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int d = wave + k * (PLACE_BLK / 64);
      if (d < 27) sl[k] = (a.mig + (int64_t)d * a.nc3)[c];
    }
  }
  // lane q < WC: the wavefront's q-th cell (count, storage start)
  uint32_t cnt = 0, beg = 0;
  if (lane < WC) {
    int qx, qy, qz;
    tile_xyz(WC * wave + lane, qx, qy, qz);
    const uint32_t c = (uint32_t)(g.cx0 + qx) + nc * ((uint32_t)(g.cy0 + qy) + nc * (uint32_t)(g.cz0 + qz));
    cnt = a.cnt[c];
    beg = (uint32_t)a.off[c];
  }
  if constexpr (NNU == 1) {
    static_assert(PLACE_BLK == 256, "one edge per thread");
    edges_lds[threadIdx.x] = a.tedge[threadIdx.x];
  }
  const float* const edges = NNU == 1 ? edges_lds : a.tedge;
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(failed)) return;  // a failed step is not applied
  const int rbase = (ox + 1) + RG * (oy + 1) + RG * RG * (oz + 1);  // ring index of own cell `lane`
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const int d = wave + k * (PLACE_BLK / 64);
    if (d < 27) next[lane * 27 + d] = offr[rbase + (d % 3 - 1) + RG * ((d / 3) % 3 - 1) + RG * RG * (d / 9 - 1)] + sl[k];
  }
  // the wavefront's cells: exclusive prefix of the counts in the lanes
  uint32_t inc = cnt;
#pragma unroll
  for (int o = 1; o < WC; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
    if (lane >= o) inc += y;
  }
  const uint32_t pre = inc - cnt;   // lanes from WC on hold the total
  const uint32_t rel = beg - pre;   // storage index of a cell's particle i: rel + i
  const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, WC - 1);
  __syncthreads();
  int ec = 0;  // the cell of the chunk's first particle
  // cell of each lane's particle of the chunk at c0, its storage index, and the lanes of its cell
  auto locate = [&](uint32_t c0, int& sc, uint32_t& p, unsigned long long& own) {
    uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)inc, ec);
    while (end <= c0) end = (uint32_t)__builtin_amdgcn_readlane((int)inc, ++ec);
    const uint32_t i = c0 + (uint32_t)lane, left = tot - c0;
    sc = ec;
    uint32_t rl = (uint32_t)__builtin_amdgcn_readlane((int)rel, ec);
    own = end - c0 >= 64u ? ~0ull : (1ull << (end - c0)) - 1ull;
    for (int q = ec + 1; q < WC && end < c0 + 64u; ++q) {
      const uint32_t b = end;  // first particle of cell q
      end = (uint32_t)__builtin_amdgcn_readlane((int)inc, q);
      const unsigned long long m = (end - c0 >= 64u ? ~0ull : (1ull << (end - c0)) - 1ull) & ~((1ull << (b - c0)) - 1ull);
      const uint32_t rq = (uint32_t)__builtin_amdgcn_readlane((int)rel, q);
      if (i >= b) {
        sc = q;
        rl = rq;
        own = m;
      }
    }
    // lanes past the end read the last particle
    p = rl + ((uint32_t)lane < left ? i : tot - 1u);
  };
  rec4 rn = {0.f, 0.f, 0.f, 0.f};
  uint32_t r2n = 0u, pn = 0u;
  uint64_t idn = 0u;
  int sn = 0;
  unsigned long long on = 0ull;
  auto request = [&]() {
    rn = rec[pn];
    if constexpr (NCHI == 2) r2n = ((Records2)(rec + a.cap))[pn];
    if constexpr (PID) idn = particle_id<0>(a, g, 0, (int64_t)pn, 0u);
  };
  // one chunk; FULL: every lane holds a particle
  auto chunk = [&](auto full, uint32_t c0) {
    constexpr bool FULL = decltype(full)::value;
    const rec4 rc = rn;
    const uint32_t r2 = r2n;
    const uint64_t id = idn;
    const int s = sn + WC * wave;
    unsigned long long peers = on;
    // the next chunk's records are requested before this chunk's stores are issued (past the end
    // the request repeats a particle of this chunk)
    if (c0 + 64u < tot) locate(c0 + 64u, sn, pn, on);
    request();
    const bool active = FULL || c0 + (uint32_t)lane < tot;
    const uint32_t w = __float_as_uint(rc.w);
    const uint32_t dc = NCHI == 1 ? w >> 24 : w >> 16;
    if constexpr (!FULL) peers &= __ballot(active);
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const bool bit = (dc >> b) & 1u;
      const unsigned long long bb = __ballot(active && bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t rin = lanes_below(peers);
    const uint32_t key = (uint32_t)s * 27u + dc;
    // ring index of the new cell: dc = (kx + 1) + 3 (ky + 1) + 9 (kz + 1) gives
    // (kx + 1) + 6 (ky + 1) + 36 (kz + 1) = dc + 3 [dc / 3] + 18 [dc / 9]
    const uint32_t t3 = (dc * 11u) >> 5, t9 = (dc * 57u) >> 9;
    const uint32_t cell = (uint32_t)((s & 3) + RG * ((s >> 2) & 3) + RG * RG * (s >> 4)) + dc + 3u * t3 + 18u * t9;
    const uint32_t b0 = next[key];
    const float4 st = stat[cell];
    if (active && rin == 0u) next[key] = b0 + (uint32_t)__popcll(peers);
    uint32_t dst = b0 + rin;
    if (active && dst >= (uint32_t)a.cap) set_flag(a.flags, FLAG_COUNT);
    dst = min(dst, (uint32_t)a.cap - 1u);
    const float u[3] = {(rc.x - st.x) * st.w, (rc.y - st.y) * st.w, (rc.z - st.z) * st.w};
    int nu[3];
    encode_nu3<NNU>(u, edges, a.vhalf, nu);
    Codes<NCHI, NNU> out;
    out.pack(NCHI == 1 ? w & 0xFFFFFFu : r2, w & 0xFFFFu, nu);
    if (active) {
      out.store(a.codes_n, a.cap, (int64_t)dst);
      if constexpr (PID) store_id(a, dst, id);
    }
  };
  if (tot > 0u) {
    locate(0u, sn, pn, on);
    request();
  }
  // whole chunks first: their stores are unconditional, so the wait for the next chunk's records
  // is for a known number of later stores and does not wait for these (with a branch around the
  // stores the compiler drains them every chunk: 1345 us for 512^3 particles)
  uint32_t c0 = 0;
  for (; c0 + 64u <= tot; c0 += 64u) chunk(std::true_type{}, c0);
  if (c0 < tot) chunk(std::false_type{}, c0);
}

template <int NCHI, int NNU, bool PID>
__global__ __launch_bounds__(PLACE_BLK) void k_place(MoveArgs a) {
  place_tile<NCHI, NNU, PID>(a, xcd_block(blockIdx.x, gridDim.x));
}

template <int NCHI, int NNU, bool PID>
__global__ __launch_bounds__(PLACE_BLK) void k_place_boxes(BoxTable<MoveArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  place_tile<NCHI, NNU, PID>(t.args[b], l - t.first[b]);
}

// ---------------------------------------------------------------------------------------------
// Link: per new cell, counts from the 27 source cells in offset order (z, y, x each -1, 0, +1),
// the slot prefix per source offset, the mean velocity and the 3-D velocity variance. The entry
// (displacement d, source cell) of the count table belongs to exactly one (new cell, source offset
// 26 - d), so the slots overwrite the counts in place, one thread per new cell.
// ---------------------------------------------------------------------------------------------
struct LinkArgs {
  uint32_t* mig;
  uint32_t* cnt_n;
  const int64_t* mom;  // the count pass's blocks per tile; load path: four planes of nc^3
  float* vc_n;
  double* dev;
  uint64_t* blk_n;
  int64_t* blk_q;
  int nc;
  int64_t nc3;
  const uint32_t* cnt_direct;  // load path: counts given directly (no migration counts)
  uint32_t* flags;
};

// the per-cell dispersion term n dev 2^20 stays below 2^54, so that the int64 sums of the 256 cells
// of a link block cannot overflow; the sum over the blocks is exact in 128 bits (k_scan_blocks, k_finalize)
constexpr double kDevTermLimit = 18014398509481984.0;  // 2^54

// Bound by memory latency, then by its 27 words read and written per cell: the 27 counts and the
// four moments of a cell are requested together (with one load waiting for the store before it, a
// 16^3 box took 15 us, now 6; 128^3 cells 139 -> 145 with the moment table, 630 MB). Cell indices fit 32 bits (nc <= 512), plane bases are uniform.
__device__ __forceinline__ void link_block(const LinkArgs& a, const unsigned blk) {
  __shared__ unsigned long long sn[LINK_BLK / 64], sq[LINK_BLK / 64];
  if (workgroup_step_failed(a.flags)) return;
  const uint32_t c = blk * LINK_BLK + threadIdx.x, nc = (uint32_t)a.nc;
  uint32_t n = 0;
  long long q = 0;
  if (c < (uint32_t)a.nc3) {
    unsigned long long m4[4];
    if (a.cnt_direct) {
      n = a.cnt_direct[c];
#pragma unroll
      for (int d = 0; d < 4; ++d) m4[d] = (unsigned long long)(a.mom + d * a.nc3)[c];
    } else {
      const uint32_t x = c % nc, y = (c / nc) % nc, z = c / (nc * nc);
      // the cell's entries in its own tile and in the tiles it lies in the ring of: beyond the lower or
      // upper face along each axis on which the cell lies at its tile's face
      const uint32_t nt = nc / T;
      uint32_t tl[3][2], rl[3][2];  // per axis: own tile and ring coordinate, neighbour's
      bool face[3];
      const uint32_t xyz[3] = {x, y, z};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const uint32_t t = xyz[d] / T, o = xyz[d] % T;
        const bool lo = o == 0, hi = o == T - 1;
        face[d] = lo || hi;
        tl[d][0] = t;
        rl[d][0] = o + 1;
        tl[d][1] = lo ? (t ? t - 1 : nt - 1) : (t + 1 < nt ? t + 1 : 0);
        rl[d][1] = lo ? T + 1 : 0;
      }
      m4[0] = m4[1] = m4[2] = m4[3] = 0;
      const ulonglong2* const tab = reinterpret_cast<const ulonglong2*>(a.mom);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int ex = e & 1, ey = (e >> 1) & 1, ez = e >> 2;
        if ((!ex || face[0]) && (!ey || face[1]) && (!ez || face[2])) {
          const uint64_t t = tl[0][ex] + nt * (tl[1][ey] + (uint64_t)nt * tl[2][ez]);
          const ulonglong2* const m = tab + (t * RC + rl[0][ex] + RG * (rl[1][ey] + RG * rl[2][ez])) * 2;
          const ulonglong2 m01 = m[0], m23 = m[1];
          m4[0] += m01.x;
          m4[1] += m01.y;
          m4[2] += m23.x;
          m4[3] += m23.y;
        }
      }
      const uint32_t xs[3] = {x ? x - 1 : nc - 1, x, x + 1 < nc ? x + 1 : 0};
      const uint32_t ys[3] = {nc * (y ? y - 1 : nc - 1), nc * y, nc * (y + 1 < nc ? y + 1 : 0)};
      const uint32_t zs[3] = {nc * nc * (z ? z - 1 : nc - 1), nc * nc * z, nc * nc * (z + 1 < nc ? z + 1 : 0)};
      uint32_t m[27];
#pragma unroll
      for (int j = 0; j < 27; ++j) m[j] = (a.mig + (int64_t)(26 - j) * a.nc3)[xs[j % 3] + ys[(j / 3) % 3] + zs[j / 9]];
#pragma unroll
      for (int j = 0; j < 27; ++j) {
        (a.mig + (int64_t)(26 - j) * a.nc3)[xs[j % 3] + ys[(j / 3) % 3] + zs[j / 9]] = n;
        n += m[j];
      }
    }
    a.cnt_n[c] = n;
    const long long s1x = (long long)m4[0], s1y = (long long)m4[1], s1z = (long long)m4[2], s2 = (long long)m4[3];
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, dev = 0.0;
    const double nd = (double)n;
    if (n > 0) {
      const double d1 = nd * 4294967296.0;
      m0 = (double)s1x / d1;
      m1 = (double)s1y / d1;
      m2 = (double)s1z / d1;
      const double d2 = nd * 16777216.0;
      const double e2 = (double)s2 / d2;
      double mm = m0 * m0;
      mm = mm + m1 * m1;
      mm = mm + m2 * m2;
      dev = e2 - mm;
      if (!(dev > 0.0)) dev = 0.0;
    }
    a.vc_n[c] = (float)m0;
    (a.vc_n + a.nc3)[c] = (float)m1;
    (a.vc_n + 2 * a.nc3)[c] = (float)m2;
    a.dev[c] = dev;
    const double term = (dev * nd) * 1048576.0;
    if (term < kDevTermLimit) {
      q = __double2ll_rn(term);
    } else {
      atomicOr(a.flags, FLAG_OVERFLOW);
      q = 0;
    }
  }
  const unsigned long long wn = wave_sum_u64(n), wq = wave_sum_u64((unsigned long long)q);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sn[wave] = wn;
    sq[wave] = wq;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tn = 0, tq = 0;
    for (int w = 0; w < LINK_BLK / 64; ++w) {
      tn += sn[w];
      tq += sq[w];
    }
    a.blk_n[blk] = tn;
    a.blk_q[blk] = (int64_t)tq;
  }
}

__global__ __launch_bounds__(LINK_BLK) void k_link(LinkArgs a) { link_block(a, xcd_block(blockIdx.x, gridDim.x)); }

__global__ __launch_bounds__(LINK_BLK) void k_link_boxes(BoxTable<LinkArgs> t) {
  const unsigned l = xcd_block(blockIdx.x, gridDim.x);
  const int b = box_of(t.first, t.nbox, l);
  link_block(t.args[b], l - t.first[b]);
}

// Nearest FP64 value (ties to even) of the unsigned 128-bit integer hi 2^64 + lo. Above 2^64 the
// value is shifted right into 64 bits with the shifted-out bits kept as a sticky lowest bit, which
// keeps the rounding to 53 bits exact; a 64-bit unsigned conversion is one rounding of the exact sum
// of its two halves.
__device__ __forceinline__ double u128_to_double(unsigned long long hi, unsigned long long lo) {
  if (hi == 0ull) return (double)lo;
  const int s = 64 - __clzll((long long)hi);  // 1 .. 64
  const unsigned long long keep = s == 64 ? hi : ((hi << (64 - s)) | (lo >> s));
  const unsigned long long lost = s == 64 ? lo : (lo & ((1ull << s) - 1ull));
  return ldexp((double)(keep | (lost != 0ull ? 1ull : 0ull)), s);
}

// the global dispersion from the 128-bit sum of its terms
__device__ __forceinline__ double global_sg2(unsigned long long hi, unsigned long long lo, int64_t n) {
  const double sg2 = u128_to_double(hi, lo) / ((3.0 * (double)n) * 1048576.0);
  return sg2 > 0.0 ? sg2 : 8.673617379884035e-19;  // 2^-60
}

// single workgroup: exclusive scan of the per-block counts; the global dispersion, the exact sum of
// the per-block int64 terms (each in [0, 2^62)) in 128 bits
struct ScanArgs {
  const uint64_t* blk_n;
  const int64_t* blk_q;
  uint64_t* blk_off;
  int64_t nblk;
  uint64_t* off_end;
  int64_t n_expect;
  double* scal;
  uint32_t* flags;
};

__device__ __forceinline__ void scan_blocks(const ScanArgs& a) {
  __shared__ unsigned long long qh[1024], ql[1024];
  __shared__ unsigned long long wtot[16];
  if (workgroup_step_failed(a.flags)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // each wavefront takes one contiguous range of the blocks, its lanes consecutive entries (the
  // loads of a wavefront coalesce); first its total count and the lanes' 128-bit dispersion sums
  const int64_t per = (a.nblk + 15) / 16;
  const int64_t b0 = min((int64_t)wave * per, a.nblk), b1 = min(b0 + per, a.nblk);
  unsigned long long s = 0, hi = 0, lo = 0;
#pragma unroll 4
  for (int64_t b = b0 + lane; b < b1; b += 64) {
    s += a.blk_n[b];
    const unsigned long long q = (unsigned long long)a.blk_q[b];
    lo += q;
    hi += lo < q ? 1ull : 0ull;
  }
  const unsigned long long ws = wave_sum_u64(s);
  if (lane == 0) wtot[wave] = ws;
  qh[tid] = hi;
  ql[tid] = lo;
  __syncthreads();
  // then the exclusive prefix of its range, 64 entries at a time, from the totals of the
  // wavefronts before it
  unsigned long long base = 0;
  for (int w = 0; w < wave; ++w) base += wtot[w];
  for (int64_t c = b0; c < b1; c += 64) {
    const int64_t b = c + lane;
    const unsigned long long n = b < b1 ? a.blk_n[b] : 0ull;
    const unsigned long long inc = wave_scan_u64(n);
    if (b < b1) a.blk_off[b] = base + inc - n;
    base += read_lane_u64(inc, 63);
  }
  for (int o = 512; o > 0; o >>= 1) {
    if (tid < o) {
      const unsigned long long l2 = ql[tid] + ql[tid + o];
      qh[tid] += qh[tid + o] + (l2 < ql[tid] ? 1ull : 0ull);
      ql[tid] = l2;
    }
    __syncthreads();
  }
  if (tid == 0) {
    unsigned long long total = 0;
    for (int w = 0; w < 16; ++w) total += wtot[w];
    *a.off_end = total;
    if ((int64_t)total != a.n_expect) atomicOr(a.flags, FLAG_COUNT);
    a.scal[0] = global_sg2(qh[0], ql[0], a.n_expect);
  }
}

__global__ __launch_bounds__(1024) void k_scan_blocks(ScanArgs a) { scan_blocks(a); }

// one workgroup per box
__global__ __launch_bounds__(1024) void k_scan_blocks_boxes(const ScanArgs* __restrict__ tab) {
  scan_blocks(tab[blockIdx.x]);
}

// Up to this many link blocks (64^3 cells) every finalize block reads all their counts and terms itself;
// above, k_scan_blocks goes before. A launch less against 16 bytes per pair of blocks from L2; link, scan
// and finalize together in us, with the scan and without: 16^3 cells 17.0 and 13.6, 48^3 20.2 and 17.5, 64^3
// 27.0 and 25.3, 96^3 87 and 92, 128^3 179 and 230.
constexpr int64_t kScanOwn = 1024;

struct FinArgs {
  const uint32_t* cnt_n;
  ScanArgs scan;
  uint64_t* off_n;
  const double* dev;
  float* vs_n;
  float* vinv;
  int64_t nc3;
  int sigma_mode;
  double sq2pi;
  const uint32_t* flags;
};

__device__ __forceinline__ void finalize_block(const FinArgs& a, const unsigned blk) {
  __shared__ uint32_t pre[LINK_BLK + 1];
  __shared__ uint32_t wsum[LINK_BLK / 64];
  __shared__ unsigned long long own[4][LINK_BLK / 64];
  if (workgroup_step_failed(a.flags)) return;
  const int64_t c = (int64_t)blk * LINK_BLK + threadIdx.x;
  const uint32_t n = (c < a.nc3) ? a.cnt_n[c] : 0u;
  const ScanArgs& g = a.scan;
  unsigned long long off;
  double sg2;
  if (g.nblk <= kScanOwn) {
    // particles before this block, all of them, and the dispersion terms' two halves: sums of at most
    // kScanOwn values of 32 bits each
    unsigned long long v[4] = {0, 0, 0, 0};
    for (uint32_t b = threadIdx.x; b < (uint32_t)g.nblk; b += LINK_BLK) {
      const unsigned long long nb = g.blk_n[b], q = (unsigned long long)g.blk_q[b];
      v[0] += b < blk ? nb : 0ull;
      v[1] += nb;
      v[2] += q & 0xffffffffull;
      v[3] += q >> 32;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned long long w = wave_sum_u64(v[k]);
      if ((threadIdx.x & 63) == 0) own[k][threadIdx.x >> 6] = w;
    }
    block_exclusive_scan(n, pre, LINK_BLK, wsum);  // (has the barriers that `own` needs)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = 0;
#pragma unroll
      for (int w = 0; w < LINK_BLK / 64; ++w) v[k] += own[k][w];
    }
    const unsigned long long lo = (v[3] << 32) + v[2];
    sg2 = global_sg2((v[3] >> 32) + (lo < v[2] ? 1ull : 0ull), lo, g.n_expect);
    off = v[0];
    const bool bad = (int64_t)v[1] != g.n_expect;
    if (blk == 0 && threadIdx.x == 0) {
      *g.off_end = v[1];
      g.scal[0] = sg2;
      if (bad) atomicOr(g.flags, FLAG_COUNT);
    }
    if (bad) return;
  } else {
    block_exclusive_scan(n, pre, LINK_BLK, wsum);
    off = g.blk_off[blk];
    sg2 = g.scal[0];
  }
  if (c >= a.nc3) return;
  a.off_n[c] = off + pre[threadIdx.x];
  double s2c = sg2;
  if (a.sigma_mode == CUBE_SIGMA_PER_CELL) {
    s2c = a.dev[c] / 3.0;
    if (n < 2 || s2c < sg2 * 9.5367431640625e-07) s2c = sg2;
  }
  const double sc = sqrt(s2c) * a.sq2pi;
  a.vs_n[c] = (float)sc;
  a.vinv[c] = (float)(1.0 / sc);
}

__global__ __launch_bounds__(LINK_BLK) void k_finalize(FinArgs a) { finalize_block(a, blockIdx.x); }

__global__ __launch_bounds__(LINK_BLK) void k_finalize_boxes(BoxTable<FinArgs> t) {
  const int b = box_of(t.first, t.nbox, blockIdx.x);
  finalize_block(t.args[b], blockIdx.x - t.first[b]);
}

// ---------------------------------------------------------------------------------------------
// Load path: host particles -> codes, stable sort by cell, moments, encode
// ---------------------------------------------------------------------------------------------
struct LoadArgs {
  const double* x;   // (n,3)
  const double* v;   // (n,3)
  int64_t n;
  int nc, nchi;
  uint32_t* key;
  uint32_t* idx;
  uint16_t* chi_tmp;  // 3 x n
  float* v_tmp;       // 3 x n
  uint32_t* cnt;
  int64_t* mom;
  int64_t nc3;
  uint32_t* flags;
};

__global__ void k_load_codes(LoadArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const int nb = 1 << (8 * a.nchi);
  int cell[3];
  for (int d = 0; d < 3; ++d) {
    double xc = a.x[3 * i + d] * 0.25;
    if (!(fabs(xc) < 1e15)) {
      atomicOr(a.flags, FLAG_NONFINITE);
      xc = 0.0;
    }
    if (xc < 0.0 || xc >= (double)a.nc) xc = xc - (double)a.nc * floor(xc / (double)a.nc);
    int c = (int)floor(xc);
    if (c >= a.nc) c -= a.nc;
    if (c < 0) c = 0;
    long long b = (long long)floor((xc - (double)c) * (double)nb);
    b = b < 0 ? 0 : (b > nb - 1 ? nb - 1 : b);
    cell[d] = c;
    a.chi_tmp[d * a.n + i] = (uint16_t)b;
  }
  const uint32_t cid = (uint32_t)(cell[0] + a.nc * (cell[1] + a.nc * cell[2]));
  a.key[i] = cid;
  a.idx[i] = (uint32_t)i;
  long long s2 = 0;
  for (int d = 0; d < 3; ++d) {
    const float vf = (float)a.v[3 * i + d];
    a.v_tmp[d * a.n + i] = vf;
    if (!(vf == vf) || fabsf(vf) >= 32768.0f) atomicOr(a.flags, FLAG_OVERFLOW);
    const double vd = (double)vf;
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.mom[d * a.nc3 + cid]),
              (unsigned long long)__double2ll_rn(vd * 4294967296.0));
    s2 += __double2ll_rn(vd * vd * 16777216.0);
  }
  atomicAdd(reinterpret_cast<unsigned long long*>(&a.mom[3 * a.nc3 + cid]), (unsigned long long)s2);
  atomicAdd(&a.cnt[cid], 1u);
}

template <int NCHI, int NNU>
__global__ void k_load_encode(const uint32_t* key_sorted, const uint32_t* idx_sorted, const uint16_t* chi_tmp,
                              const float* v_tmp, int64_t n, void* codes_out, int64_t cap,
                              const float* vc, const float* vinv, int64_t nc3, const float* edges,
                              int vhalf, void* pid_out, int pid_bytes) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int64_t src = idx_sorted[j];
  const int64_t c = key_sorted[j];
  const float inv = vinv[c];
  int ch[3], nu[3];
  float u[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    ch[d] = (int)chi_tmp[d * n + src];
    u[d] = (v_tmp[d * n + src] - vc[d * nc3 + c]) * inv;
  }
  encode_nu3<NNU>(u, edges, vhalf, nu);
  Codes<NCHI, NNU> w;
  w.set(ch, nu);
  w.store(codes_out, cap, j);
  // the ID of a loaded particle is its index in the input
  if (pid_bytes == 8) static_cast<uint64_t*>(pid_out)[j] = (uint64_t)src;
  else if (pid_bytes == 4) static_cast<uint32_t*>(pid_out)[j] = (uint32_t)src;
}

// Between the packed words and the checkpoint's planes (chi: 3 planes of n codes, nu: 3 planes of n)
template <int NCHI, int NNU>
__global__ __launch_bounds__(256) void k_unpack_codes(const void* codes, int64_t cap, int64_t n, void* chi, void* nu) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
    Codes<NCHI, NNU> w;
    w.load(codes, cap, j);
    int ch[3], nv[3];
    w.chi(ch);
    w.nu(nv);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      static_cast<chi_t<NCHI>*>(chi)[d * n + j] = (chi_t<NCHI>)ch[d];
      static_cast<nu_t<NNU>*>(nu)[d * n + j] = (nu_t<NNU>)nv[d];
    }
  }
}

template <int NCHI, int NNU>
__global__ __launch_bounds__(256) void k_pack_codes(const void* chi, const void* nu, int64_t n, void* codes, int64_t cap) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
    int ch[3], nv[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      ch[d] = (int)static_cast<const chi_t<NCHI>*>(chi)[d * n + j];
      nv[d] = (int)static_cast<const nu_t<NNU>*>(nu)[d * n + j];
    }
    Codes<NCHI, NNU> w;
    w.set(ch, nv);
    w.store(codes, cap, j);
  }
}

// IDs 0 .. n-1 in storage order
__global__ void k_pid_iota(void* pid, int pid_bytes, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  if (pid_bytes == 8) static_cast<uint64_t*>(pid)[j] = (uint64_t)j;
  else static_cast<uint32_t*>(pid)[j] = (uint32_t)j;
}

// ---------------------------------------------------------------------------------------------
// White noise: Philox4x32-10 (Salmon et al. 2011) keyed by (seed, lattice index), Box-Muller.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void philox_round(uint32_t* c, uint32_t k0, uint32_t k1) {
  const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
  const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
  const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
  const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
  const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
  c[0] = n0;
  c[1] = lo1;
  c[2] = n2;
  c[3] = lo0;
}

// grid: x covers one z plane of n^2 points, y = z (keeps each grid dimension below 2^32 items)
__global__ void k_noise(float* out, int n, int64_t pitch_f, uint64_t seed) {
  const int64_t ixy = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (ixy >= (int64_t)n * n) return;
  const int64_t i = (int64_t)blockIdx.y * n * n + ixy;
  uint32_t c[4] = {(uint32_t)i, (uint32_t)((uint64_t)i >> 32), 0u, 0u};
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    philox_round(c, k0, k1);
  }
  const double u0 = ((double)c[0] + 0.5) * 2.3283064365386962890625e-10;
  const double u1 = ((double)c[1] + 0.5) * 2.3283064365386962890625e-10;
  const double w = sqrt(-2.0 * log(u0)) * cos(6.283185307179586 * u1);
  const int64_t x = i % n, y = (i / n) % n, z = i / ((int64_t)n * n);
  out[(z * n + y) * pitch_f + x] = (float)w;
}

// Amplitude per |n|^2 of the initial conditions, the host cosmology's expressions term by term. Before,
// the host filled the table and the transforms waited for it: 196609 entries (512^3 particles) 9 ms, now
// 30 us; bound by the latencies of FP64 log1p and pow. Both sides' errors together stay below 32 units
// of 2^-53 of the value; entries within 2^-42 of a rounding boundary (2 in 10^6) are left to the host, so
// that the table is the same bit for bit.
__global__ __launch_bounds__(256) void k_ic_table(ICTable c, float* __restrict__ tab, uint32_t* __restrict__ near_list) {
  const int64_t n2 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n2 >= c.ntab) return;
  if (n2 == 0) {
    tab[0] = 0.0f;
    return;
  }
  const double k = 2.0 * 3.14159265358979323846 * sqrt((double)n2) / c.box;
  const double q = k / c.omh;
  const double t1 = log1p(2.34 * q) / (2.34 * q);
  const double q1 = 16.1 * q, q2 = 5.46 * q, q3 = 6.71 * q;
  const double poly = 1.0 + 3.89 * q + q1 * q1 + q2 * q2 * q2 + (q3 * q3) * (q3 * q3);
  const double t = t1 * pow(poly, -0.25);
  const double pk = c.amp * pow(k, c.ns) * t * t;
  const double amp = sqrt(c.np3 * pk * c.di * c.di / (c.box * c.box * c.box));
  const double v = amp * c.nm / (2.0 * 3.14159265358979323846 * (double)n2 * c.np3);
  const double e = v * 2.2737367544323206e-13;  // 2^-42
  tab[n2] = (float)v;
  if (!((float)(v - e) == (float)(v + e))) {
    const uint32_t i = atomicAdd(&near_list[0], 1u);
    if (i < kICNear) near_list[1 + i] = (uint32_t)n2;
  }
}

}  // namespace

// =============================================================================================
// host launchers
// =============================================================================================
#define CUBE_XV_DISPATCH(nchi, nnu, CALL)                                     \
  do {                                                                        \
    if ((nchi) == 1 && (nnu) == 1) CALL(1, 1);                                \
    else if ((nchi) == 1 && (nnu) == 2) CALL(1, 2);                           \
    else if ((nchi) == 2 && (nnu) == 1) CALL(2, 1);                           \
    else CALL(2, 2);                                                          \
  } while (0)

// side of the deposit's columns in coarse cells: 8, where the ring is 36 cells to 64 and a workgroup of 16
// wavefronts shares its planes; 4 in boxes of at most 32 cells a side, which have too few columns of 8
// to fill the chip (16^3 cells 27 -> 14 us; with 64^3 cells columns of 4 take 232 us, of 8 113)
static int deposit_dtx(const Sim& s) { return s.nc <= 32 ? 4 : 8; }

// the deposit's arguments for the state of parity cur, and its grid (columns x z chunks)
static DepArgs deposit_args(const Sim& s, int cur, dim3* grid) {
  DepArgs a;
  a.codes = s.codes[cur];
  a.cnt = s.cnt[cur];
  a.off = s.off[cur];
  a.cap = s.capacity;
  a.mesh = s.mesh;
  a.pitch_f = (int64_t)s.mesh_plan.row_floats();
  a.nm = s.nm;
  a.nc = s.nc;
  const int dtx = deposit_dtx(s), cols = (s.nc / dtx) * (s.nc / dtx);
  // z chunks: about 2048 workgroups of 16 wavefronts are four rounds of the chip, and a chunk of zc layers
  // reads zc + 2 (512^3 cells: 749 us; in 4096 chunks 809, in 8192 956); at least 4 layers, 2 in columns of 4
  int nchunk = dtx == 8 ? 2048 / cols : s.nc / 2;
  const int thin = dtx == 8 ? 4 : 2;
  nchunk = nchunk < 1 ? 1 : (nchunk > s.nc / thin ? s.nc / thin : nchunk);
  a.zc = (s.nc + nchunk - 1) / nchunk;
  nchunk = (s.nc + a.zc - 1) / a.zc;
  a.inv_mean = (double)s.nm * (double)s.nm * (double)s.nm / ((double)s.n * ldexp(1.0, 3 * (8 * s.nchi - 1)));
  a.flags = s.flags;
  *grid = dim3((unsigned)cols, (unsigned)nchunk);
  return a;
}

// the deposit kernel NAME for columns of dtx cells and nchi-byte positions
#define CUBE_DEP(NAME, GRID, ARG)                                                          \
  do {                                                                                     \
    if (dtx == 4 && nchi == 1) NAME<1, 4, 256><<<GRID, 256, 0, st>>>(ARG);                  \
    else if (dtx == 4) NAME<2, 4, 256><<<GRID, 256, 0, st>>>(ARG);                          \
    else if (nchi == 1) NAME<1, 8, 1024><<<GRID, 1024, 0, st>>>(ARG);                       \
    else NAME<2, 8, 1024><<<GRID, 1024, 0, st>>>(ARG);                                      \
  } while (0)

void launch_deposit(Sim& s, hipStream_t st) {
  dim3 grid;
  const DepArgs a = deposit_args(s, s.cur, &grid);
  const int dtx = deposit_dtx(s), nchi = s.nchi;
  CUBE_DEP(k_deposit, grid, a);
  CUBE_HIP(hipGetLastError());
}

// arguments of the link, block-scan and finalize kernels that build state nxt
static LinkArgs link_args(const Sim& s, int nxt, const uint32_t* cnt_direct) {
  LinkArgs l;
  l.mig = s.mig;
  l.cnt_n = s.cnt[nxt];
  l.mom = s.mom;
  l.vc_n = s.vc[nxt];
  l.dev = s.dev;
  l.blk_n = s.blk_n;
  l.blk_q = s.blk_q;
  l.nc = s.nc;
  l.nc3 = s.nc3;
  l.cnt_direct = cnt_direct;
  l.flags = s.flags;
  return l;
}

static ScanArgs scan_args(const Sim& s, int nxt) {
  return ScanArgs{s.blk_n, s.blk_q, s.blk_off, s.nblk, s.off[nxt] + s.nc3, s.n, s.scal, s.flags};
}

static FinArgs fin_args(const Sim& s, int nxt) {
  FinArgs f;
  f.cnt_n = s.cnt[nxt];
  f.scan = scan_args(s, nxt);
  f.off_n = s.off[nxt];
  f.dev = s.dev;
  f.vs_n = s.vs[nxt];
  f.vinv = s.vinv;
  f.nc3 = s.nc3;
  f.sigma_mode = s.p.sigma_mode;
  f.sq2pi = std::sqrt(2.0 / M_PI);
  f.flags = s.flags;
  return f;
}

static void link_scan_finalize(Sim& s, int nxt, const uint32_t* cnt_direct, hipStream_t st) {
  k_link<<<(unsigned)s.nblk, LINK_BLK, 0, st>>>(link_args(s, nxt, cnt_direct));
  CUBE_HIP(hipGetLastError());
  if (s.nblk > kScanOwn) {
    k_scan_blocks<<<1, 1024, 0, st>>>(scan_args(s, nxt));
    CUBE_HIP(hipGetLastError());
  }
  k_finalize<<<(unsigned)s.nblk, LINK_BLK, 0, st>>>(fin_args(s, nxt));
  CUBE_HIP(hipGetLastError());
}

__global__ void k_step_end(uint32_t* flags, int* step, uint32_t code) {
  if (threadIdx.x != 0) return;
  if (step) {
    code = (uint32_t)step[0] + 2u;
    step[0] += 1;
  }
  if (flags[0] != 0u && flags[1] == 0u) flags[1] = code;
}

void launch_step_end(Sim& s, hipStream_t st, uint32_t code, bool dev_sched) {
  k_step_end<<<1, 64, 0, st>>>(s.flags, dev_sched ? s.step_dev : nullptr, code);
  CUBE_HIP(hipGetLastError());
}

// flags[0] |= f, when step is null or the device step counter equals `at`
__global__ void k_raise_flag(uint32_t* flags, const int* step, int at, uint32_t f) {
  if (threadIdx.x == 0 && (!step || step[0] == at)) flags[0] |= f;
}

void launch_raise_flag(Sim& s, hipStream_t st, uint32_t f, bool dev_sched, int at) {
  k_raise_flag<<<1, 64, 0, st>>>(s.flags, dev_sched ? s.step_dev : nullptr, at, f);
  CUBE_HIP(hipGetLastError());
}

// whether a step's scatter places the count pass's records (k_place) instead of recomputing the
// move: when the record buffer is there; a poll limit other than the default asks for the ordered
// scatter it belongs to
static bool use_records(const Sim& s) { return step_records(s) != nullptr; }

// the move passes' arguments from the state of parity cur to the other (no step maxima, no
// initial-condition fields)
static MoveArgs move_args(const Sim& s, int cur, float kfac, float dfac, bool dev_sched) {
  const int nxt = cur ^ 1;
  MoveArgs a{};
  a.codes = s.codes[cur];
  a.cnt = s.cnt[cur];
  a.off = s.off[cur];
  a.vc = s.vc[cur];
  a.vs = s.vs[cur];
  a.codes_n = s.codes[nxt];
  a.off_n = s.off[nxt];
  a.vc_n = s.vc[nxt];
  a.vinv = s.vinv;
  a.cap = s.capacity;
  a.mesh = s.mesh;
  a.pitch_f = (int64_t)s.mesh_plan.row_floats();
  a.nm = s.nm;
  a.nc = s.nc;
  a.nt = s.nc / T;
  a.nc3 = s.nc3;
  a.kf = kfac;
  a.df = dfac;
  a.tdec = s.tdec;
  a.tedge = s.tedge;
  a.vhalf = (s.vm - 1) / 2;
  a.mig = s.mig;
  a.mom = s.mom;
  a.flags = s.flags;
  a.kd = dev_sched ? s.sched_dev : nullptr;
  a.kstep = dev_sched ? s.step_dev : nullptr;
  a.pid = s.pid[cur];
  a.pid_n = s.pid[nxt];
  a.pid_bytes = s.pid_bytes;
  a.amax = nullptr;
  a.rec = reinterpret_cast<float4*>(step_records(s));
  a.turn_limit = s.turn_limit;
  return a;
}

// whether a step's recomputing scatter uses the gradient tile: move_variant 1 and 2, -1 when there are
// at least half as many particles as fine cells
static bool tile_scatter(const Sim& s) {
  const bool dense = 2 * s.n >= (int64_t)s.nm * s.nm * s.nm;
  return s.move_variant < 0 ? dense : (s.move_variant == 1 || s.move_variant == 2);
}

void launch_move(Sim& s, int mode, float kfac, float dfac, float* const* psi, float vfac, hipStream_t st,
                 hipEvent_t* evs, bool dev_sched) {
  const int nxt = s.cur ^ 1;
  MoveArgs a = move_args(s, s.cur, kfac, dfac, dev_sched);
  // step maxima for adaptive time steps (a small fill kernel clears them: no memset node in
  // captured graphs, although adaptive simulations are never captured)
  a.amax = (mode == 0 && s.amax) ? s.amax : nullptr;
  if (a.amax) {
    k_clear_u32<<<1, 64, 0, st>>>(s.amax, 2);
    CUBE_HIP(hipGetLastError());
  }
  if (mode == 2) {
    a.psi0 = psi[0];
    a.psi1 = psi[1];
    a.psi2 = psi[2];
    a.lat_pitch_f = (int64_t)s.lat_plan.row_floats();
    a.np = s.np;
    a.q = s.np / s.nc;
    a.vfac = vfac;
    a.lunit = (float)(2.0 / (double)a.q);
  }
  const unsigned grid = (unsigned)((int64_t)a.nt * a.nt * a.nt);
#define CUBE_COUNT(X, V)                                                                        \
  do {                                                                                          \
    if (mode == 0 && a.amax) k_count<X, V, 0, true><<<grid, CNTH, 0, st>>>(a);                   \
    else if (mode == 0) k_count<X, V, 0><<<grid, CNTH, 0, st>>>(a);                              \
    else if (mode == 1) k_count<X, V, 1><<<grid, CNTH, 0, st>>>(a);                              \
    else k_count<X, V, 2><<<grid, CNTH, 0, st>>>(a);                                             \
  } while (0)
#define CUBE_SCATTER(X, V)                                                                      \
  do {                                                                                          \
    if (mode != 2 && a.rec && a.pid_bytes) k_place<X, V, true><<<grid, PLACE_BLK, 0, st>>>(a);   \
    else if (mode != 2 && a.rec) k_place<X, V, false><<<grid, PLACE_BLK, 0, st>>>(a);            \
    else if (mode == 0 && tile_scatter(s)) k_scatter_dense<X, V><<<grid, 1024, 0, st>>>(a);                   \
    else if (mode == 0) k_move_scatter<X, V, 0, 512><<<grid, 512, 0, st>>>(a);            \
    else if (mode == 1) k_move_scatter<X, V, 1, 256><<<grid, 256, 0, st>>>(a);            \
    else k_move_scatter<X, V, 2, 256><<<grid, 256, 0, st>>>(a);                           \
  } while (0)
  if (evs) CUBE_HIP(hipEventRecord(evs[0], st));
  CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_COUNT);
  CUBE_HIP(hipGetLastError());
  if (evs) CUBE_HIP(hipEventRecord(evs[1], st));
  link_scan_finalize(s, nxt, nullptr, st);
  if (evs) CUBE_HIP(hipEventRecord(evs[2], st));
  CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_SCATTER);
  CUBE_HIP(hipGetLastError());
  if (evs) CUBE_HIP(hipEventRecord(evs[3], st));
#undef CUBE_COUNT
#undef CUBE_SCATTER
  s.cur = nxt;
}

// ---- ensemble steps: one launch per stage over every box ---------------------------------------
size_t EnsembleStep::put(const void* p, size_t bytes) {
  const size_t off = (staged.size() + 255) & ~(size_t)255;
  staged.resize(off + bytes);
  if (bytes) std::memcpy(staged.data() + off, p, bytes);
  return off;
}

void EnsembleStep::upload() {
  if (dbase || staged.empty()) return;
  CUBE_HIP(hipMalloc(&dbase, staged.size()));
  CUBE_HIP(hipMemcpy(dbase, staged.data(), staged.size(), hipMemcpyHostToDevice));
}

EnsembleStep::~EnsembleStep() {
  if (dbase) (void)hipFree(dbase);
}

namespace {

// a staged per-box argument table with the first workgroup of each box
struct StagedBoxes {
  size_t args, first;
  int nbox;
  unsigned blocks;  // workgroups of the launch
};

template <class A>
StagedBoxes stage_boxes(EnsembleStep& es, const std::vector<A>& args, const std::vector<uint32_t>& per_box,
                        int threads) {
  std::vector<uint32_t> first(1, 0u);
  uint64_t t = 0;
  for (uint32_t b : per_box) {
    t += b;
    first.push_back((uint32_t)t);
  }
  if (!fits_dispatch(t, (uint64_t)threads)) throw Error{CUBE_E_INVALID, "ensemble too large for one launch per stage"};
  return StagedBoxes{es.put(args), es.put(first), (int)args.size(), (unsigned)t};
}

template <class A>
BoxTable<A> table_of(const EnsembleStep* e, const StagedBoxes& g) {
  return BoxTable<A>{e->at<A>(g.args), e->at<uint32_t>(g.first), g.nbox};
}

struct EndArgs {
  uint32_t* flags;
  int* step;
};

// k_step_end of every box (device step counters), one thread per box
__global__ void k_step_end_boxes(const EndArgs* __restrict__ tab, int nbox) {
  const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (b >= nbox) return;
  uint32_t* flags = tab[b].flags;
  int* step = tab[b].step;
  const uint32_t code = (uint32_t)step[0] + 2u;
  step[0] += 1;
  if (flags[0] != 0u && flags[1] == 0u) flags[1] = code;
}

}  // namespace

void ensemble_deposit(EnsembleStep& es, const std::vector<Sim*>& boxes) {
  const EnsembleStep* e = &es;
  for (int nchi = 1; nchi <= 2; ++nchi)
    for (int dtx : {4, 8}) {
      std::vector<DepArgs> args;
      std::vector<uint32_t> per;
      for (Sim* s : boxes) {
        if (s->nchi != nchi || deposit_dtx(*s) != dtx) continue;
        dim3 g;
        args.push_back(deposit_args(*s, s->cur, &g));
        per.push_back(g.x * g.y);
      }
      if (args.empty()) continue;
      const StagedBoxes g = stage_boxes(es, args, per, dtx == 4 ? 256 : 1024);
      es.launches.push_back([e, g, nchi, dtx](hipStream_t st) {
        const BoxTable<DepArgs> t = table_of<DepArgs>(e, g);
        CUBE_DEP(k_deposit_boxes, g.blocks, t);
        CUBE_HIP(hipGetLastError());
      });
    }
}

void ensemble_move(EnsembleStep& es, const std::vector<Sim*>& boxes) {
  const EnsembleStep* e = &es;
  // one pass over the boxes grouped by codec and kernel (0 per-corner gradient, 1 gradient tile, 2 the
  // scatter from records, 3 that with particle IDs)
  auto pass = [&](bool scatter) {
    for (int xv = 0; xv < 4; ++xv)
      for (int tile = 0; tile <= 3; ++tile) {
        const int nchi = 1 + (xv >> 1), nnu = 1 + (xv & 1);
        std::vector<MoveArgs> args;
        std::vector<uint32_t> per;
        for (Sim* s : boxes) {
          const int kern = scatter ? (use_records(*s) ? (s->pid_bytes ? 3 : 2) : (tile_scatter(*s) ? 1 : 0)) : 0;
          if (s->nchi != nchi || s->nnu != nnu || kern != tile) continue;
          args.push_back(move_args(*s, s->cur, 0.0f, 0.0f, true));
          const int64_t nt = s->nc / T;
          per.push_back((uint32_t)(nt * nt * nt));
        }
        if (args.empty()) continue;
        // The count pass's workgroups are twice as wide as those of the per-corner scatter, which bounds an
        // ensemble at 2^23 tiles: from 2^22 on it takes two launches
        const int threads = scatter ? (tile >= 2 ? PLACE_BLK : (tile ? 1024 : 512)) : CNTH;
        uint64_t tiles = 0;
        for (uint32_t b : per) tiles += b;
        if (!scatter && !fits_dispatch(tiles, 512)) throw Error{CUBE_E_INVALID, "ensemble too large for one launch per stage"};
        const std::vector<size_t> runs = scatter ? std::vector<size_t>{0, per.size()} : box_runs(per, (uint64_t)threads);
        for (size_t i = 0; i + 1 < runs.size(); ++i) {
          const size_t b0 = runs[i], b1 = runs[i + 1];
          const StagedBoxes g = stage_boxes(es, std::vector<MoveArgs>(args.begin() + b0, args.begin() + b1),
                                            std::vector<uint32_t>(per.begin() + b0, per.begin() + b1), threads);
          es.launches.push_back([e, g, nchi, nnu, tile, scatter](hipStream_t st) {
            const BoxTable<MoveArgs> t = table_of<MoveArgs>(e, g);
#define CUBE_PASS(X, V)                                                                                 \
  do {                                                                                                  \
    if (tile == 3) k_place_boxes<X, V, true><<<g.blocks, PLACE_BLK, 0, st>>>(t);                         \
    else if (tile == 2) k_place_boxes<X, V, false><<<g.blocks, PLACE_BLK, 0, st>>>(t);                   \
    else if (tile && scatter) k_scatter_dense_boxes<X, V><<<g.blocks, 1024, 0, st>>>(t);                   \
    else if (scatter) k_move_scatter_boxes<X, V, 0, 512><<<g.blocks, 512, 0, st>>>(t);            \
    else k_count_boxes<X, V><<<g.blocks, CNTH, 0, st>>>(t);                                              \
  } while (0)
            CUBE_XV_DISPATCH(nchi, nnu, CUBE_PASS);
#undef CUBE_PASS
            CUBE_HIP(hipGetLastError());
          });
        }
      }
  };
  pass(false);
  // link, block scan and finalize of every box
  std::vector<LinkArgs> la;
  std::vector<ScanArgs> sa;
  std::vector<FinArgs> fa;
  std::vector<uint32_t> per;
  for (Sim* s : boxes) {
    const int nxt = s->cur ^ 1;
    la.push_back(link_args(*s, nxt, nullptr));
    if (s->nblk > kScanOwn) sa.push_back(scan_args(*s, nxt));
    fa.push_back(fin_args(*s, nxt));
    per.push_back((uint32_t)s->nblk);
  }
  const StagedBoxes gl = stage_boxes(es, la, per, LINK_BLK);
  const StagedBoxes gf = stage_boxes(es, fa, per, LINK_BLK);
  const size_t os = es.put(sa);
  const unsigned nscan = (unsigned)sa.size();
  es.launches.push_back([e, gl, gf, os, nscan](hipStream_t st) {
    k_link_boxes<<<gl.blocks, LINK_BLK, 0, st>>>(table_of<LinkArgs>(e, gl));
    CUBE_HIP(hipGetLastError());
    if (nscan) {
      k_scan_blocks_boxes<<<nscan, 1024, 0, st>>>(e->at<ScanArgs>(os));
      CUBE_HIP(hipGetLastError());
    }
    k_finalize_boxes<<<gf.blocks, LINK_BLK, 0, st>>>(table_of<FinArgs>(e, gf));
    CUBE_HIP(hipGetLastError());
  });
  pass(true);
}

void ensemble_step_end(EnsembleStep& es, const std::vector<Sim*>& boxes) {
  std::vector<EndArgs> t;
  for (Sim* s : boxes) t.push_back(EndArgs{s->flags, s->step_dev});
  const size_t ot = es.put(t);
  const int nbox = (int)boxes.size();
  const EnsembleStep* e = &es;
  es.launches.push_back([e, ot, nbox](hipStream_t st) {
    k_step_end_boxes<<<(unsigned)((nbox + 63) / 64), 64, 0, st>>>(e->at<EndArgs>(ot), nbox);
    CUBE_HIP(hipGetLastError());
  });
}

void launch_load(Sim& s, const double* dx, const float* /*unused*/, int64_t n, hipStream_t st) {
  // scratch for the load path
  const int nxt = s.cur ^ 1;
  uint32_t* key = static_cast<uint32_t*>(s.dmalloc(sizeof(uint32_t) * n * 4));
  uint32_t* idx = key + n;
  uint32_t* key2 = key + 2 * n;
  uint32_t* idx2 = key + 3 * n;
  uint16_t* chi_tmp = static_cast<uint16_t*>(s.dmalloc(sizeof(uint16_t) * 3 * n));
  float* v_tmp = static_cast<float*>(s.dmalloc(sizeof(float) * 3 * n));
  CUBE_HIP(hipMemsetAsync(s.cnt[nxt], 0, sizeof(uint32_t) * s.nc3, st));
  CUBE_HIP(hipMemsetAsync(s.mom, 0, sizeof(int64_t) * 4 * s.nc3, st));
  LoadArgs a;
  a.x = dx;
  a.v = dx + 3 * n;
  a.n = n;
  a.nc = s.nc;
  a.nchi = s.nchi;
  a.key = key;
  a.idx = idx;
  a.chi_tmp = chi_tmp;
  a.v_tmp = v_tmp;
  a.cnt = s.cnt[nxt];
  a.mom = s.mom;
  a.nc3 = s.nc3;
  a.flags = s.flags;
  if (n > 0) {
    k_load_codes<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(a);
    CUBE_HIP(hipGetLastError());
  }
  // stable sort of (cell id, input index) by cell id
  uint32_t *ks = key, *is = idx;
  sort_pairs_by_key(s, key, idx, key2, idx2, n, (uint32_t)(s.nc3 - 1), st, &ks, &is);
  link_scan_finalize(s, nxt, s.cnt[nxt], st);
#define CUBE_ENC(X, V)                                                                                       \
  k_load_encode<X, V><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(ks, is, chi_tmp, v_tmp, n, s.codes[nxt],  \
                                                                   s.capacity, s.vc[nxt], s.vinv, \
                                                                   s.nc3, s.tedge, (s.vm - 1) / 2, \
                                                                   s.pid[nxt], s.pid_bytes)
  if (n > 0) {
    CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_ENC);
    CUBE_HIP(hipGetLastError());
  }
#undef CUBE_ENC
  CUBE_HIP(hipStreamSynchronize(st));
  s.dfree(v_tmp);
  s.dfree(chi_tmp);
  s.dfree(key);
  s.cur = nxt;
}

// where the checkpoint's planes are staged: in the other state buffer (scratch between steps), the
// wider codes first so that each plane is aligned to its code
void staged_planes(const Sim& s, void** chi, void** nu) {
  char* const w = static_cast<char*>(s.codes[s.cur ^ 1]);
  const bool chi_first = s.nchi >= s.nnu;
  *chi = chi_first ? w : w + (size_t)3 * s.n * s.nnu;
  *nu = chi_first ? w + (size_t)3 * s.n * s.nchi : w;
}

// workgroups of the two conversions, which go round the particles: a launch holds less than 2^32 threads
static unsigned pack_blocks(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, 65536); }

void launch_unpack_codes(Sim& s, hipStream_t st) {
  if (s.n == 0) return;
  void *chi, *nu;
  staged_planes(s, &chi, &nu);
#define CUBE_UNPACK(X, V) \
  k_unpack_codes<X, V><<<pack_blocks(s.n), 256, 0, st>>>(s.codes[s.cur], s.capacity, s.n, chi, nu)
  CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_UNPACK);
#undef CUBE_UNPACK
  CUBE_HIP(hipGetLastError());
}

void launch_pack_codes(Sim& s, hipStream_t st) {
  if (s.n == 0) return;
  void *chi, *nu;
  staged_planes(s, &chi, &nu);
#define CUBE_PACK(X, V) \
  k_pack_codes<X, V><<<pack_blocks(s.n), 256, 0, st>>>(chi, nu, s.n, s.codes[s.cur], s.capacity)
  CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_PACK);
#undef CUBE_PACK
  CUBE_HIP(hipGetLastError());
}

void launch_pid_iota(Sim& s, hipStream_t st) {
  if (!s.pid_bytes || s.n == 0) return;
  k_pid_iota<<<(unsigned)((s.n + 255) / 256), 256, 0, st>>>(s.pid[s.cur], s.pid_bytes, s.n);
  CUBE_HIP(hipGetLastError());
}

// largest |v|^2 of the decoded state (the velocity bound of the first adaptive steps): one thread
// per particle, its cell found by bisection in the cell offsets
template <int NCHI, int NNU>
__global__ void k_state_speed(const void* codes, const uint64_t* off, const float* vc, const float* vs,
                              const float* tdec, int64_t n, int64_t cap, int64_t nc3, int vhalf, uint32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float vv = 0.0f;
  if (i < n) {
    int64_t lo = 0, hi = nc3;  // the cell c with off[c] <= i < off[c + 1]
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (off[mid] <= (uint64_t)i) lo = mid;
      else hi = mid;
    }
    Codes<NCHI, NNU> w;
    w.load(codes, cap, i);
    int nv[3];
    w.nu(nv);
    float v[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      int c = nv[d];
      c = c < -vhalf ? -vhalf : (c > vhalf ? vhalf : c);
      v[d] = __builtin_fmaf(vs[lo], tdec[c + vhalf], vc[d * nc3 + lo]);
    }
    vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
  }
  vv = wave_max(vv);
  if ((threadIdx.x & 63) == 0 && vv > 0.0f) atomicMax(out, __float_as_uint(vv));
}

float launch_state_speed2(Sim& s, hipStream_t st) {
  k_clear_u32<<<1, 64, 0, st>>>(s.amax, 2);
  CUBE_HIP(hipGetLastError());
  if (s.n > 0) {
    const unsigned grid = (unsigned)((s.n + 255) / 256);
    const int vh = (s.vm - 1) / 2;
#define CUBE_SPEED(X, V)                                                                                              \
  k_state_speed<X, V><<<grid, 256, 0, st>>>(s.codes[s.cur], s.off[s.cur], s.vc[s.cur], s.vs[s.cur], s.tdec, s.n,         \
                                            s.capacity, s.nc3, vh, s.amax)
    CUBE_XV_DISPATCH(s.nchi, s.nnu, CUBE_SPEED);
#undef CUBE_SPEED
    CUBE_HIP(hipGetLastError());
  }
  uint32_t bits = 0;
  CUBE_HIP(hipMemcpyAsync(&bits, s.amax, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
  CUBE_HIP(hipStreamSynchronize(st));
  float f;
  std::memcpy(&f, &bits, sizeof(f));
  return f;
}

// 1-byte coarse density (Sec. 2.1): min(count, 255) per cell
__global__ void k_counts_u8(const uint32_t* cnt, int64_t nc3, uint8_t* rho1) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nc3) return;
  const uint32_t v = cnt[c];
  rho1[c] = (uint8_t)(v < 255u ? v : 255u);
}

int64_t launch_counts_u8(Sim& s, uint8_t* rho1, uint32_t* over, hipStream_t st) {
  const uint32_t* cnt = s.cnt[s.cur];
  k_counts_u8<<<(unsigned)((s.nc3 + 255) / 256), 256, 0, st>>>(cnt, s.nc3, rho1);
  CUBE_HIP(hipGetLastError());
  // the true counts of the cells marked 255, in cell order (a stable selection)
  return select_at_least_255(s, cnt, s.nc3, over, st);
}

void launch_ic_table(const ICTable& c, float* tab, uint32_t* near_list, hipStream_t st) {
  CUBE_HIP(hipMemsetAsync(near_list, 0, sizeof(uint32_t), st));
  k_ic_table<<<(unsigned)((c.ntab + 255) / 256), 256, 0, st>>>(c, tab, near_list);
  CUBE_HIP(hipGetLastError());
}

void launch_noise(const FFTPlan& pl, float* out, uint64_t seed, hipStream_t st) {
  const int64_t plane = (int64_t)pl.n * pl.n;
  const dim3 grid((unsigned)((plane + 255) / 256), (unsigned)pl.n);
  k_noise<<<grid, 256, 0, st>>>(out, pl.n, (int64_t)pl.row_floats(), seed);
  CUBE_HIP(hipGetLastError());
}

}  // namespace cube
