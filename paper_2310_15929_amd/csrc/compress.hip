// Compression of n:m-pruned weights (Section 4, step 1): kept values + 2 bits of index per kept
// value, written both in the canonical row-major form and in the order the sparse-MFMA kernels
// stream (the layout is documented in include/esparse.h).  Pure data movement: HBM-bound.
#include <algorithm>

#include "common.h"

// state[K] |= 1 : perm is not a bijection; the kernels behind then leave the outputs alone.  host_flags (pinned host memory,
// written only where there is something to report): 1 = a group does not keep exactly n, 2 = perm is not a bijection
__global__ void k_perm_count(const int32_t* __restrict__ perm, long long K, int* __restrict__ state, int* __restrict__ host_flags) {
  long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= K) return;
  const int c = perm[p];
  if (c < 0 || c >= K || atomicAdd(&state[c], 1) != 0) {
    atomicOr(&state[K], 1);
    host_flags[1] = 1;
  }
}

// ---- 2:4 ----------------------------------------------------------------------------------------
// One unit = (row, 16 re-ordered channels): 4 groups, 8 kept values, 16 index bits.
// wrow points at the row's weights in ORIGINAL channel order (global memory or an LDS copy).
// Units beyond N or K (padding of the native tiling) are written as zeros.
__device__ __forceinline__ void compress_unit_2_4(const uint16_t* wrow, const uint8_t* __restrict__ mrow /*mask row or null*/,
                                                  const int32_t* __restrict__ perm, bool live, long long row, long long ch,
                                                  long long K, long long Kp, uint16_t* __restrict__ values,
                                                  uint32_t* __restrict__ meta, uint16_t* __restrict__ nvalues,
                                                  uint16_t* __restrict__ nmeta, int* __restrict__ host_flags) {
  uint16_t kept[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t bits = 0;
  int nk = 0;  // kept values in this unit (8 unless the unit is cut by K or is padding)
  const long long p0 = ch * 16;
  if (live && p0 < K) {
    const int ngroups = (int)((K - p0) >= 16 ? 4 : (K - p0) / 4);
    uint32_t mk4[4] = {0, 0, 0, 0};
    if (mrow) {
      if (ngroups == 4 && (K & 15) == 0) {
        const uint4 mv = *reinterpret_cast<const uint4*>(mrow + p0);
        mk4[0] = mv.x; mk4[1] = mv.y; mk4[2] = mv.z; mk4[3] = mv.w;
      } else {
        for (int g = 0; g < ngroups; g++) mk4[g] = *reinterpret_cast<const uint32_t*>(mrow + p0 + g * 4);
      }
    }
    bool bad = false;
#pragma unroll
    for (int g = 0; g < 4; g++) {
      if (g >= ngroups) break;
      uint16_t w[4];
      int c4[4];
      if (perm) {
        const int4 pv = *reinterpret_cast<const int4*>(perm + p0 + g * 4);
        c4[0] = pv.x; c4[1] = pv.y; c4[2] = pv.z; c4[3] = pv.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; i++) c4[i] = (int)(p0 + g * 4 + i);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) w[i] = wrow[c4[i]];
      uint32_t mk;  // one byte per position, non-zero = kept
      if (mrow) {
        mk = mk4[g];
      } else {
        // keep the non-zero weights, topped up with the lowest-position zeros
        mk = 0;
        int nz = 0;
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (w[i] & 0x7fffu) {
            mk |= 1u << (8 * i);
            nz++;
          }
        if (nz > 2) bad = true;
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (nz < 2 && !((mk >> (8 * i)) & 0xffu)) {
            mk |= 1u << (8 * i);
            nz++;
          }
      }
      int cnt = 0;
#pragma unroll
      for (int i = 0; i < 4; i++)
        if ((mk >> (8 * i)) & 0xffu) {
          if (cnt < 2) {
            // nk = 2 g + cnt : compile-time g, so the two slots are selected without dynamic indexing
            if (cnt == 0) kept[2 * g] = w[i];
            else kept[2 * g + 1] = w[i];
            bits |= (uint32_t)i << (2 * (2 * g + cnt));
          }
          cnt++;
        }
      if (cnt != 2) bad = true;  // the call reports EBADMASK; the slot layout stays well-formed
      nk = 2 * g + 2;
    }
    if (bad) host_flags[0] = 1;
    // canonical: values[row][ch*8 .. ch*8+nk), index half-words
    if (values) {
      uint16_t* dst = values + row * (K / 2) + ch * 8;
      if (nk == 8 && ((K / 2) % 8 == 0)) {
        uint4 v;
        v.x = kept[0] | ((uint32_t)kept[1] << 16);
        v.y = kept[2] | ((uint32_t)kept[3] << 16);
        v.z = kept[4] | ((uint32_t)kept[5] << 16);
        v.w = kept[6] | ((uint32_t)kept[7] << 16);
        *reinterpret_cast<uint4*>(dst) = v;
      } else {
#pragma unroll
        for (int i = 0; i < 8; i++)
          if (i < nk) dst[i] = kept[i];
      }
    }
    if (meta) {
      // uint32 words per row: ceil(K/32); this unit is half-word (ch & 1) of word ch / 2
      uint16_t* m16 = reinterpret_cast<uint16_t*>(meta + row * ((K / 2 + 15) / 16));
      m16[ch] = (uint16_t)bits;
      if (p0 + 16 >= K && (ch & 1) == 0) m16[ch + 1] = 0;  // unused half of the row's last word
    }
  }
  if (nvalues) {
    const long long nchunk = Kp / 16;
    const long long rt = row >> 4, ks = ch >> 2;
    const int r = (int)(row & 15), ga = (int)(ch & 3);
    uint4 v;
    v.x = kept[0] | ((uint32_t)kept[1] << 16);
    v.y = kept[2] | ((uint32_t)kept[3] << 16);
    v.z = kept[4] | ((uint32_t)kept[5] << 16);
    v.w = kept[6] | ((uint32_t)kept[7] << 16);
    reinterpret_cast<uint4*>(nvalues)[((rt * (nchunk / 4) + ks) * 4 + ga) * 16 + r] = v;
    // index unit order [rt][ks/4][ga][r][ks%4]
    nmeta[(((rt * (nchunk / 16) + ks / 4) * 4 + ga) * 16 + r) * 4 + (ks & 3)] = (uint16_t)bits;
  }
}

// Generic form: one thread per unit, weights gathered from global memory (any K).
__global__ void __launch_bounds__(256) k_compress_2_4(const uint16_t* __restrict__ W, const uint8_t* __restrict__ mask,
                                                       const int32_t* __restrict__ perm, long long N, long long K, long long Np,
                                                       long long Kp, uint16_t* __restrict__ values, uint32_t* __restrict__ meta,
                                                       uint16_t* __restrict__ nvalues, uint16_t* __restrict__ nmeta,
                                                       const int* __restrict__ bad_perm, int* __restrict__ host_flags) {
  if (bad_perm && *bad_perm) return;
  const long long nchunk = Kp / 16;
  long long u = (long long)blockIdx.x * 256 + threadIdx.x;
  if (u >= Np * nchunk) return;
  // thread order = native unit order, so the native stores are coalesced
  const int r = (int)(u & 15), ga = (int)((u >> 4) & 3);
  const long long t = u >> 6;
  const long long ks = t % (nchunk / 4), rt = t / (nchunk / 4);
  const long long row = rt * 16 + r, ch = ks * 4 + ga;
  const bool live = row < N;
  compress_unit_2_4(W + (live ? row : 0) * K, mask ? mask + (live ? row : 0) * K : nullptr, perm, live, row, ch, K, Kp, values,
                    meta, nvalues, nmeta, host_flags);
}

// ---- 4:8 ----------------------------------------------------------------------------------------
// One thread per (row, group of 8) of the padded matrix: 4 kept values + one bitmap byte.
// Native form (what the 4:8 product streams; same size and unit numbering as the 2:4 one): the group
// of row 16 rt + r that covers channels 64 ks + 32 h + 8 g .. + 8 is the A operand of lane 16 g + r of
// the dense 16x16x32 instruction for half-step h of step ks.  Its 4 kept values (8 bytes) sit at byte
// 8 h of the 16-byte unit (rt nks + ks) 64 + lane; its pattern code is byte h of the 16-bit word at the place
// where the 2:4 form keeps that lane's index half for step ks.  The pattern code of a group is the index of its
// bitmap among the 70 bitmaps with four bits set, in ascending order (the product kernels look their byte-permute
// selectors up by it, and 70 entries can be replicated in LDS where 256 cannot).  Padding rows and channels hold
// zero values and code 0.
__device__ __forceinline__ uint32_t pattern_code_4_8(uint32_t bm) {
  // sum over the set positions p_1 < p_2 < ... of C(p_j, j): the bitmaps below bm that first differ from it at p_j
  uint32_t code = 0;
  int j = 0;
#pragma unroll
  for (int e = 0; e < 8; e++)
    if ((bm >> e) & 1u) {
      j++;
      int c = 1;
      for (int t = 0; t < j; t++) c = c * (e - t) / (t + 1);
      code += (uint32_t)c;
    }
  return code;
}

__global__ void __launch_bounds__(256) k_compress_4_8(const uint16_t* __restrict__ W, const uint8_t* __restrict__ mask,
                                                       const int32_t* __restrict__ perm, long long N, long long K, long long Np,
                                                       long long Kp, uint16_t* __restrict__ values, uint8_t* __restrict__ meta,
                                                       unsigned char* __restrict__ nvalues, uint8_t* __restrict__ nmeta,
                                                       const int* __restrict__ bad_perm, int* __restrict__ host_flags) {
  if (bad_perm && *bad_perm) return;
  const long long ng = K / 8, ngp = Kp / 8;
  long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= Np * ngp) return;
  const long long row = e / ngp, g = e % ngp;
  uint16_t kept[4] = {0, 0, 0, 0};
  uint32_t bm = 0;
  if (row < N && g < ng) {
    uint16_t w[8];
    uint8_t mk[8];
    int nz = 0;
#pragma unroll
    for (int i = 0; i < 8; i++) {
      long long p = g * 8 + i;
      long long c = perm ? perm[p] : p;
      w[i] = W[row * K + c];
      mk[i] = mask ? (mask[row * K + p] ? 1 : 0) : ((w[i] & 0x7fffu) ? 1 : 0);
      nz += mk[i];
    }
    if (!mask) {
      if (nz > 4) host_flags[0] = 1;
#pragma unroll
      for (int i = 0; i < 8; i++)
        if (nz < 4 && !mk[i]) {
          mk[i] = 1;
          nz++;
        }
    }
    if (nz != 4) host_flags[0] = 1;
    int nk = 0;
#pragma unroll
    for (int i = 0; i < 8; i++)
      if (mk[i] && nk < 4) {
        kept[nk++] = w[i];
        bm |= 1u << i;
      }
    if (values) {
      uint2 v;
      v.x = kept[0] | ((uint32_t)kept[1] << 16);
      v.y = kept[2] | ((uint32_t)kept[3] << 16);
      *reinterpret_cast<uint2*>(values + row * (K / 2) + g * 4) = v;
    }
    if (meta) meta[row * ng + g] = (uint8_t)bm;
  }
  if (nvalues) {
    const long long nks = Kp / 64;
    const long long rt = row >> 4, ks = g >> 3;
    const int r = (int)(row & 15), h = (int)((g >> 2) & 1), gg = (int)(g & 3);
    const int lane = gg * 16 + r;
    uint2 v;
    v.x = kept[0] | ((uint32_t)kept[1] << 16);
    v.y = kept[2] | ((uint32_t)kept[3] << 16);
    *reinterpret_cast<uint2*>(nvalues + ((rt * nks + ks) * 64 + lane) * 16 + 8 * h) = v;
    nmeta[(((rt * (nks / 4) + ks / 4) * 64 + lane) * 4 + (ks & 3)) * 2 + h] = (uint8_t)pattern_code_4_8(bm);
  }
}

// ---- both patterns, rows in LDS -------------------------------------------------------------------
// A workgroup copies RB whole rows of W into LDS with coalesced loads and gathers the permuted channels from there, so HBM
// sees W exactly once, in order.  Needs 2 K RB bytes of LDS.  A thread takes one row and, of 256 channels, the 16 (2:4) or
// 8 (4:8) channels at quarter ga of each 64-channel step: four 16-byte units of the native form and its 8 bytes of indices.
// Four neighbouring lanes (ga) exchange their indices, so that the canonical ones leave 8 bytes at a time as well - one unit
// per thread wrote both in pieces of 2 bytes.  The mask is on its way before the rows have arrived.  The lanes of a wave are
// 4 quarters x rows, so that both value forms leave in runs of 64 to 128 bytes.
// HBM-bound: 11008 x 4096 fp16, both forms (237 MB): 2:4 66 -> 56 us (4.2 TB/s; a copy runs at 5.1).  Whole calls: 126 -> 88
// us, 4:8 229 -> 121; 9216 x 36864 2:4 1067 -> 599, 4096 x 11008 4:8 383 -> 136.
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
  switch (lane) {
    case 0: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x00, 0xf, 0xf, true);
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x55, 0xf, 0xf, true);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xaa, 0xf, 0xf, true);
    default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xff, 0xf, 0xf, true);
  }
#else
  (void)lane;
  return v;
#endif
}

// element i without dynamic indexing
__device__ __forceinline__ int element(const int (&v)[4], int i) {
  const int a = (i & 1) ? v[1] : v[0], b = (i & 1) ? v[3] : v[2];
  return (i & 2) ? b : a;
}
__device__ __forceinline__ int element(const int (&v)[8], int i) {
  const int a = (i & 1) ? v[1] : v[0], b = (i & 1) ? v[3] : v[2], c = (i & 1) ? v[5] : v[4], d = (i & 1) ? v[7] : v[6];
  const int e = (i & 2) ? b : a, f = (i & 2) ? d : c;
  return (i & 4) ? f : e;
}

// four mask bytes (non-zero = kept) as four bits
__device__ __forceinline__ uint32_t kept_by_mask(uint32_t mk) {
  const uint32_t on = ((((mk & 0x7f7f7f7fu) + 0x7f7f7f7fu) | mk) & 0x80808080u) >> 7;  // bits 0, 8, 16, 24
  return (on * 0x10204080u) >> 28;  // 2^28, 2^21, 2^14, 2^7 bring them to bits 28, 29, 30, 31
}
// without a mask: the non-zero weights, topped up with the lowest-position zeros; false if there are more than n
template <int NKEEP, int MG>
__device__ __forceinline__ bool kept_by_value(const uint16_t* wrow, const int (&c)[MG], uint32_t& bm) {
  bm = 0;
#pragma unroll
  for (int i = 0; i < MG; i++) bm |= (wrow[c[i]] & 0x7fffu) ? 1u << i : 0u;
  const bool ok = __popc(bm) <= NKEEP;
#pragma unroll
  for (int i = 0; i < MG; i++) bm |= __popc(bm) < NKEEP ? 1u << i : 0u;
  return ok;
}

template <int NKEEP, int MG, bool MASK, bool PERM, int THREADS>
__global__ void __launch_bounds__(THREADS) k_compress_rows(const uint16_t* __restrict__ W, const uint8_t* __restrict__ mask,
                                                        const int32_t* __restrict__ perm, long long N, long long K, long long Np,
                                                        long long first_row /*multiple of 128*/, int RB, int nkb /*256-channel steps*/, uint16_t* __restrict__ values, void* __restrict__ meta,
                                                        unsigned char* __restrict__ native, const int* __restrict__ bad_perm,
                                                        int* __restrict__ host_flags) {
  constexpr int GU = MG == 4 ? 4 : 2;       // groups per 16-byte unit
  extern __shared__ uint2 s_w2[];           // [RB][K / 4] groups of 4 weights
  __shared__ uint8_t s_code[256];           // 4:8: pattern code of a bitmap
  if (bad_perm && *bad_perm) return;
  const int tid = threadIdx.x;
  // the 16 / RB workgroups of a row tile are numbered 8 apart: they run on one XCD at about the same time, and their pieces of
  // the native form leave its L2 as whole lines
  const int per = 16 / RB;
  const long long row0 = first_row + ((long long)(blockIdx.x / (8 * per)) * 8 + blockIdx.x % 8) * 16 + (blockIdx.x / 8) % per * RB;
  if (row0 >= Np) return;
  const int k4 = (int)(K / 4);
  const int work = RB * nkb * 4;
  const uint16_t* s_w = reinterpret_cast<const uint16_t*>(s_w2);
  // a thread's places: e = ((kb RB) + r) 4 + ga
  uint4 mk[4];
  const bool wide_mask = (K & 15) == 0;  // 16 bytes at once (2:4), 8 (4:8)
  auto load_mask = [&](int e) {
    const int ga = e & 3, t = e >> 2, r = t % RB, kb = t / RB;
    const long long row = row0 + r;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      mk[j] = uint4{0u, 0u, 0u, 0u};
      if (row >= N) continue;
      const uint8_t* mrow = mask + row * K;
      if (MG == 4) {
        const long long p0 = (long long)((kb * 4 + j) * 4 + ga) * 16;
        if (wide_mask && p0 + 16 <= K) {
          mk[j] = *reinterpret_cast<const uint4*>(mrow + p0);
        } else {
          const uint32_t* m4 = reinterpret_cast<const uint32_t*>(mrow + p0);
          if (p0 < K) mk[j].x = m4[0];
          if (p0 + 4 < K) mk[j].y = m4[1];
          if (p0 + 8 < K) mk[j].z = m4[2];
          if (p0 + 12 < K) mk[j].w = m4[3];
        }
      } else {
        const long long p0 = (long long)(kb * 4 + j) * 64 + 8 * ga;  // rows of a multiple of 8 bytes
        if (p0 < K) {
          const uint2 v = *reinterpret_cast<const uint2*>(mrow + p0);
          mk[j].x = v.x;
          mk[j].y = v.y;
        }
        if (p0 + 32 < K) {
          const uint2 v = *reinterpret_cast<const uint2*>(mrow + p0 + 32);
          mk[j].z = v.x;
          mk[j].w = v.y;
        }
      }
    }
  };
  if (MASK && tid < work) load_mask(tid);
  {
    const long long left = N - row0;
    const int nr = (int)(left < RB ? (left > 0 ? left : 0) : RB);
    const uint2* src = reinterpret_cast<const uint2*>(W) + row0 * k4;
    for (int c = tid; c < nr * k4; c += THREADS) s_w2[c] = src[c];
  }
  if (MG == 8 && tid < 256) {
    // sum over the set positions p_1 < p_2 < ... of C(p_j, j): the bitmaps below this one that first differ from it at p_j
    int code = 0, j = 0;
    for (int e = 0; e < 8; e++)
      if ((tid >> e) & 1) {
        j++;
        int c = 1;
        for (int t = 0; t < j; t++) c = c * (e - t) / (t + 1);
        code += c;
      }
    s_code[tid] = (uint8_t)code;
  }
  __syncthreads();
  bool bad = false;
  for (int e = tid; e < work; e += THREADS) {
    if (MASK && e != tid) load_mask(e);
    const int ga = e & 3, t = e >> 2, r = t % RB, kb = t / RB;
    const long long row = row0 + r;
    if (row >= Np) continue;
    const bool live = row < N;
    const uint16_t* wrow = s_w + (size_t)r * K;
    // no branches up to the stores, so that the loads of the permutation and the reads of the weights of several groups are
    // under way together; what lies past K or N reads channel 0 and becomes zero
    uint4 unit[4];
    uint32_t idx[4];  // 2:4: 16 index bits of the unit; 4:8: two bitmaps
#pragma unroll
    for (int j = 0; j < 4; j++) {
      uint16_t kept[8];
      idx[j] = 0;
#pragma unroll
      for (int u = 0; u < GU; u++) {
        const int p0 = MG == 4 ? ((kb * 4 + j) * 4 + ga) * 16 + 4 * u : (kb * 4 + j) * 64 + 32 * u + 8 * ga;
        const bool in = live && p0 < (int)K;
        const int ps = p0 < (int)K ? p0 : 0;
        int c[MG];
#pragma unroll
        for (int h = 0; h < MG / 4; h++) {
          int4 pv = int4{ps + 4 * h, ps + 4 * h + 1, ps + 4 * h + 2, ps + 4 * h + 3};
          if (PERM) pv = *reinterpret_cast<const int4*>(perm + ps + 4 * h);
          c[4 * h] = pv.x;
          c[4 * h + 1] = pv.y;
          c[4 * h + 2] = pv.z;
          c[4 * h + 3] = pv.w;
        }
        uint32_t bm;
        bool ok = true;
        if (MASK && MG == 4) bm = kept_by_mask(u == 0 ? mk[j].x : u == 1 ? mk[j].y : u == 2 ? mk[j].z : mk[j].w);
        else if (MASK) bm = kept_by_mask(u == 0 ? mk[j].x : mk[j].z) | (kept_by_mask(u == 0 ? mk[j].y : mk[j].w) << 4);
        else ok = kept_by_value<NKEEP, MG>(wrow, c, bm);
        ok = ok && __popc(bm) == NKEEP;
        bad = bad || (in && !ok);  // the call reports EBADMASK; what it writes then is not used
        // only the kept weights are read: their positions, lowest first
        uint32_t rest = bm;
#pragma unroll
        for (int q = 0; q < NKEEP; q++) {
          const int i = (__ffs((int)rest) - 1) & (MG - 1);
          rest &= rest - 1;
          kept[u * NKEEP + q] = in ? wrow[element(c, i)] : (uint16_t)0;
          if (MG == 4) idx[j] |= in ? (uint32_t)i << (4 * u + 2 * q) : 0u;
        }
        if (MG == 8) idx[j] |= in ? bm << (8 * u) : 0u;
      }
      unit[j] = uint4{kept[0] | ((uint32_t)kept[1] << 16), kept[2] | ((uint32_t)kept[3] << 16), kept[4] | ((uint32_t)kept[5] << 16),
                      kept[6] | ((uint32_t)kept[7] << 16)};
    }
    if (native) {
      const long long rt = row >> 4, nks = (long long)nkb * 4;
      const int rr = (int)(row & 15);
      uint4* nv = reinterpret_cast<uint4*>(native);
#pragma unroll
      for (int j = 0; j < 4; j++) nv[((rt * nks + kb * 4 + j) * 4 + ga) * 16 + rr] = unit[j];
      uint32_t m[4];
#pragma unroll
      for (int j = 0; j < 4; j++) m[j] = MG == 4 ? idx[j] : (uint32_t)s_code[idx[j] & 0xffu] | ((uint32_t)s_code[idx[j] >> 8] << 8);
      reinterpret_cast<uint2*>(native + Np * (long long)nkb * 256)[((rt * nkb + kb) * 4 + ga) * 16 + rr] = uint2{m[0] | (m[1] << 16), m[2] | (m[3] << 16)};
    }
    if (values && live) {
      uint16_t* vrow = values + row * (K / 2);
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (MG == 4) {
          const long long p0 = (long long)((kb * 4 + j) * 4 + ga) * 16;
          if (p0 + 16 <= K && wide_mask) {
            *reinterpret_cast<uint4*>(vrow + p0 / 2) = unit[j];
          } else {
            const uint32_t v[4] = {unit[j].x, unit[j].y, unit[j].z, unit[j].w};
#pragma unroll
            for (int g = 0; g < 4; g++)
              if (p0 + 4 * g < K) *reinterpret_cast<uint32_t*>(vrow + p0 / 2 + 2 * g) = v[g];
          }
        } else {
          const long long p0 = (long long)(kb * 4 + j) * 64 + 8 * ga;
          if (p0 < K) *reinterpret_cast<uint2*>(vrow + p0 / 2) = uint2{unit[j].x, unit[j].y};
          if (p0 + 32 < K) *reinterpret_cast<uint2*>(vrow + p0 / 2 + 16) = uint2{unit[j].z, unit[j].w};
        }
      }
    }
    if (meta && live) {
      // lane ga takes step 4 kb + ga: the four lanes' indices of that step
      const uint32_t lo = idx[0] | (idx[1] << 16), hi = idx[2] | (idx[3] << 16);
      uint32_t h[4];  // 16 bits of each lane
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const uint32_t ql = quad_bcast(lo, q), qh = quad_bcast(hi, q);
        h[q] = ((ga & 2 ? qh : ql) >> (16 * (ga & 1))) & 0xffffu;
      }
      const long long ks = (long long)kb * 4 + ga;
      if (MG == 4) {  // unit q of the step
        const long long words = (K / 2 + 15) / 16;
        uint32_t* dst = reinterpret_cast<uint32_t*>(meta) + row * words + ks * 2;
        if (ks * 2 < words) dst[0] = h[0] | (h[1] << 16);
        if (ks * 2 + 1 < words) dst[1] = h[2] | (h[3] << 16);
      } else {  // byte 4 u + q: group of 8 number 8 ks + 4 u + q
        uint8_t* dst = reinterpret_cast<uint8_t*>(meta) + row * (K / 8) + ks * 8;
        const uint2 v = uint2{(h[0] & 0xffu) | ((h[1] & 0xffu) << 8) | ((h[2] & 0xffu) << 16) | (h[3] << 24),
                              (h[0] >> 8) | ((h[1] >> 8) << 8) | ((h[2] >> 8) << 16) | ((h[3] >> 8) << 24)};
        if ((K & 63) == 0) {
          if (ks * 64 < K) *reinterpret_cast<uint2*>(dst) = v;
        } else {
#pragma unroll
          for (int b = 0; b < 8; b++)
            if ((ks * 8 + b) * 8 < K) dst[b] = (uint8_t)((b < 4 ? v.x : v.y) >> (8 * (b & 3)));
        }
      }
    }
  }
  if (bad) host_flags[0] = 1;
}

int esp_compress_device(esparse_ctx* ctx, const void* Wv, const uint8_t* mask, const int32_t* perm, long long N,
                        long long K, int dtype, int n, int m, void* values_out, void* meta_out, void* native_out) {
  (void)dtype;  // both dtypes are 16-bit patterns here
  (void)n;
  hipStream_t st = ctx->stream;
  Scratch scratch(ctx);
  // what the kernels report: in host memory, so that neither clearing nor reading it takes a place in the stream
  volatile int* flags = reinterpret_cast<volatile int*>(esp_host_stage(ctx, 2 * sizeof(int)));
  if (!flags) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
  flags[0] = flags[1] = 0;
  int* host_flags = const_cast<int*>(flags);
  int* bad_perm = nullptr;
  if (perm) {
    int* state = scratch.get<int>(K + 1);
    if (!state) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
    ESP_HIP(ctx, hipMemsetAsync(state, 0, (K + 1) * 4, st));
    hipLaunchKernelGGL(k_perm_count, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, perm, K, state, host_flags);
    ESP_HIP(ctx, hipGetLastError());
    bad_perm = state + K;
  }
  const uint16_t* W = reinterpret_cast<const uint16_t*>(Wv);
  const long long Np = native_out ? esp_round_up(N, 16) : N;
  const long long Kp = esp_round_up(K, 256);
  const size_t row_bytes = (size_t)K * 2;
  // rows per workgroup, a power of two: four workgroups of four rows per CU up to 5120 channels, two down to one row where
  // 64 KiB hold no more, and what fits beyond
  int RB = row_bytes <= 159 * 1024 ? 1 : 0;
  while (RB && RB < 4 && 2 * RB * row_bytes <= (row_bytes <= 64 * 1024 ? 64 * 1024 : 159 * 1024)) RB *= 2;
  if (RB) {
    const size_t smem = (size_t)RB * row_bytes;
    // a launch has fewer than 2^32 threads (more are cut off without an error): 2^31 at most, in several launches if need be
    const long long per = 16 / RB, tiles = (Np + 15) / 16, tiles_at_once = (1ll << 21) / per;
#define LAUNCH_THREADS(NK, MGv, MASKv, PERMv, THv)                                                                             \
  do {                                                                                                                         \
    if (smem > 64 * 1024)                                                                                                      \
      ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_compress_rows<NK, MGv, MASKv, PERMv, THv>),            \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));                                \
    for (long long t0 = 0; t0 < tiles; t0 += tiles_at_once)                                                                    \
      hipLaunchKernelGGL((k_compress_rows<NK, MGv, MASKv, PERMv, THv>),                                                        \
                         dim3((unsigned)((std::min(tiles - t0, tiles_at_once) + 7) / 8 * 8 * per)), dim3(THv), smem, st, W, mask, perm, N, K, Np, \
                         t0 * 16, RB, (int)(Kp / 256), reinterpret_cast<uint16_t*>(values_out), meta_out,                      \
                         reinterpret_cast<unsigned char*>(native_out), bad_perm, host_flags);                                  \
  } while (0)
// 16 waves per CU whatever the LDS leaves room for
#define LAUNCH_ROWS(NK, MGv, MASKv, PERMv)                                       \
  do {                                                                           \
    if (smem <= 40 * 1024) LAUNCH_THREADS(NK, MGv, MASKv, PERMv, 256);           \
    else if (smem <= 79 * 1024) LAUNCH_THREADS(NK, MGv, MASKv, PERMv, 512);      \
    else LAUNCH_THREADS(NK, MGv, MASKv, PERMv, 1024);                            \
  } while (0)
#define LAUNCH_PATTERN(NK, MGv)                      \
  do {                                               \
    if (mask && perm) LAUNCH_ROWS(NK, MGv, true, true); \
    else if (mask) LAUNCH_ROWS(NK, MGv, true, false);   \
    else if (perm) LAUNCH_ROWS(NK, MGv, false, true);   \
    else LAUNCH_ROWS(NK, MGv, false, false);            \
  } while (0)
    if (m == 4) LAUNCH_PATTERN(2, 4);
    else LAUNCH_PATTERN(4, 8);
#undef LAUNCH_PATTERN
#undef LAUNCH_THREADS
#undef LAUNCH_ROWS
  } else if (m == 4) {
    uint16_t* nmeta = native_out ? reinterpret_cast<uint16_t*>(reinterpret_cast<unsigned char*>(native_out) + (size_t)Np * Kp) : nullptr;
    const long long Nt = esp_round_up(N, 16), units = Nt * (Kp / 16);  // numbered by row tiles, whatever is written
    hipLaunchKernelGGL(k_compress_2_4, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, W, mask, perm, N, K, Nt, Kp,
                       reinterpret_cast<uint16_t*>(values_out), reinterpret_cast<uint32_t*>(meta_out),
                       reinterpret_cast<uint16_t*>(native_out), nmeta, bad_perm, host_flags);
  } else {
    const long long Kq = native_out ? Kp : K;
    const long long groups = Np * (Kq / 8);
    uint8_t* nmeta = native_out ? reinterpret_cast<uint8_t*>(native_out) + (size_t)Np * Kp : nullptr;
    hipLaunchKernelGGL(k_compress_4_8, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st, W, mask, perm, N, K, Np, Kq,
                       reinterpret_cast<uint16_t*>(values_out), reinterpret_cast<uint8_t*>(meta_out),
                       reinterpret_cast<unsigned char*>(native_out), nmeta, bad_perm, host_flags);
  }
  ESP_HIP(ctx, hipGetLastError());
  ESP_HIP(ctx, hipStreamSynchronize(st));
  scratch.idle();
  if (flags[1]) return esp_fail(ctx, ESPARSE_EBADPERM, "perm is not a bijection on [0, %lld)", K);
  if (flags[0]) return esp_fail(ctx, ESPARSE_EBADMASK, "a group of %d does not keep exactly %d weights", m, n);
  return ESPARSE_OK;
}

// ---- dense re-tiling (the dense GEMM streams W the same way the sparse one streams its values) ----
// unit = (row, 8 channels) = 16 bytes; order [row/16][chunk/4][chunk%4][row%16]; zero padded.
__global__ void __launch_bounds__(256) k_dense_pack(const uint16_t* __restrict__ W, long long N, long long K, long long Np,
                                                     long long Kp, uint4* __restrict__ out) {
  const long long nchunk = Kp / 8;
  long long u = (long long)blockIdx.x * 256 + threadIdx.x;
  if (u >= Np * nchunk) return;
  const int r = (int)(u & 15), g = (int)((u >> 4) & 3);
  const long long t = u >> 6;
  const long long ks = t % (nchunk / 4), rt = t / (nchunk / 4);
  const long long row = rt * 16 + r, k0 = (ks * 4 + g) * 8;
  uint16_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (row < N)
    for (int e = 0; e < 8; e++)
      if (k0 + e < K) v[e] = W[row * K + k0 + e];
  uint4 o;
  o.x = v[0] | ((uint32_t)v[1] << 16);
  o.y = v[2] | ((uint32_t)v[3] << 16);
  o.z = v[4] | ((uint32_t)v[5] << 16);
  o.w = v[6] | ((uint32_t)v[7] << 16);
  out[u] = o;
}

int esp_dense_pack_device(esparse_ctx* ctx, const void* W, long long N, long long K, int dtype, void* packed) {
  (void)dtype;
  const long long Np = esp_round_up(N, 16), Kp = esp_round_up(K, 256);
  const long long units = Np * (Kp / 8);
  hipLaunchKernelGGL(k_dense_pack, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, ctx->stream,
                     reinterpret_cast<const uint16_t*>(W), N, K, Np, Kp, reinterpret_cast<uint4*>(packed));
  ESP_HIP(ctx, hipGetLastError());
  return ESPARSE_OK;
}
