// Token permutation (Sec. 3.3 / 3.4) fused with block-mean pooling (Sec. 3.2, eqs. 5-6),
// the key-major re-tiling of V for the attention kernel, and the inverse permutation.
// Both kernels are pure HBM traffic: every row moves as 16-byte vectors, a group of
// d/8 neighbouring lanes moving one whole row.
#include "rf2_internal.h"

namespace {

typedef unsigned short u16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Every row is read once and written once: non-temporal accesses keep the stream from displacing
// other data in the caches on its way (measured on the 720p layer: loads alone -4 %, stores alone
// +0.5 %, both -9 % of the time).  Layers small beside the Infinity Cache (256 MB) are better kept in it: the attention
// finds qp, kp, vp there, and the inputs, which the program has just made, are.  Measured on image layers of 4,096 tokens, the
// buffers of three layers in turn (us, layer / permutation alone; bytes read and written):
//   non-temporal     stores kept      both kept
//   70.5 /  -        67.4 /  -        64.6 /  -         10 heads,  63 MB
//   76.6 / 15.3      75.2 / 15.8      73.4 / 12.6       12 heads,  75 MB
//   91.2 / 19.3      88.6 / 18.8      89.6 / 21.8       16 heads, 101 MB
//   145  / 28.7      140  / 28.5      140  / 31.3       24 heads, 151 MB
//   169  / 36.6      165  / 38.5      166  / 40.5       32 heads, 201 MB
// Both are kept up to 80 MiB (84 MB), stores alone up to 160 MiB (168 MB; beyond, the permutation itself gets slower, up to 8 %).
// Bytes read and written, rows of the last, partly filled blocks included.
constexpr int64_t KEEP_ALL = (int64_t)80 << 20, KEEP_STORES = (int64_t)160 << 20;
// The inverse permutation reads what the attention has just written (non-temporal -> kept loads, us, token-major and not: 50 MB
// 13.8 -> 9.6, 84 MB 17.1 -> 13.8, 118 MB 22.0 -> 19.0, 166 MB 35.3 -> 26.8, 258 MB 49.8 -> 51.4, 335 MB 115 -> 121): up to 192 MiB (201 MB).
constexpr int64_t KEEP_UNPERMUTE = (int64_t)192 << 20;

template <bool KEEP>
__device__ __forceinline__ uint4 ld_stream(const uint4* p) {
  const u32x4* const from = reinterpret_cast<const u32x4*>(p);
  const u32x4 v = KEEP ? *from : __builtin_nontemporal_load(from);
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool KEEP>
__device__ __forceinline__ void st_stream(uint4* p, uint4 v) {
  const u32x4 w = {v.x, v.y, v.z, v.w};
  if constexpr (KEEP) *reinterpret_cast<u32x4*>(p) = w;
  else __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// One workgroup gathers one block of BLK permuted rows of Q (IS_K = false) or K (true),
// writes them in permuted order and reduces their column sums to the block mean.
// Q rows stay row-major; a K block is written as BLK/64 operand parts [D/8][64][8]: with
// KH = BLK/2, the 16-byte chunk c of block row r lands in part (r % KH) / 32 at chunk slot
// c*64 + (r / KH)*32 + r % 32 -- the order in which the attention kernel's matrix-core
// operand reads walk it (a part holds one 32-key tile of each key half).
template <int D>
using pool_rows = float[256 / (D / 8)][D + 1];
template <int D, int BLK, bool IS_K, int KEEP>
__device__ __forceinline__ void permute_pool_block(
    const uint4* __restrict__ x, uint4* __restrict__ xp, float* __restrict__ mean, const int32_t* __restrict__ perm,
    int n_blocks, int last_valid, int heads, const rf2_strides& st, int blk, int bh, pool_rows<D>& part) {
  constexpr int CH = D / 8;          // 16-byte chunks per row
  constexpr int RG = 256 / CH;       // rows moved per pass
  const uint4* __restrict__ src = x + ((bh / heads) * st.batch + (bh % heads) * st.head) * CH;
  uint4* __restrict__ dst = xp + ((size_t)bh * n_blocks + blk) * BLK * CH;
  // Q: CH neighbouring lanes move one row (row-major stores).  K: 8 neighbouring lanes move half a row
  // (one 128-byte line) and a wavefront covers 8 rows x 8 chunks, so that its stores of a chunk
  // column (8 consecutive rows x 16 bytes in the operand layout) are whole 128-byte lines too.
  int c = threadIdx.x % CH, rg = threadIdx.x / CH;
  if constexpr (IS_K && CH == 16) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    c = (lane & 7) + 8 * (wave & 1);
    rg = (lane >> 3) + 8 * (wave >> 1);
  }

  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int r = rg; r < BLK; r += RG) {
    const int n = perm[blk * BLK + r];
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (n >= 0) v = ld_stream<KEEP == 2>(&src[(size_t)n * st.token * CH + c]);
    constexpr int KH = BLK / 2;
    const int kslot = ((r % KH) / 32 * CH + c) * 64 + (r / KH) * 32 + r % 32;
    st_stream<KEEP >= 1>(&dst[IS_K ? kslot : r * CH + c], v);
    acc[0] += bf16_lo(v.x); acc[1] += bf16_hi(v.x);
    acc[2] += bf16_lo(v.y); acc[3] += bf16_hi(v.y);
    acc[4] += bf16_lo(v.z); acc[5] += bf16_hi(v.z);
    acc[6] += bf16_lo(v.w); acc[7] += bf16_hi(v.w);
  }
  if (mean == nullptr) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) part[rg][c * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll
    for (int g = 0; g < RG; ++g) s += part[g][threadIdx.x];   // fixed order: bit-reproducible
    const int cnt = (blk == n_blocks - 1) ? last_valid : BLK;
    mean[((size_t)bh * n_blocks + blk) * D + threadIdx.x] = s / (float)cnt;
  }
}

// Position inside a 16-key group of the key-major V tile -> key offset (see rf2.h).
__device__ __forceinline__ int rho(int r) { return (r & 3) | ((r & 4) << 1) | ((r & 8) >> 1); }

// One workgroup gathers the 64 permuted rows of V that make up one operand part into LDS and writes
// the part [8][D][8] of the attention kernel's second product (16 KiB or 8 KiB, contiguous).
// Storage position s of a key inside its block: each 16-key group is listed in the order
// 0-3, 8-11, 4-7, 12-15.  With KH = BLK/2, position s goes to part (s % KH) / 32, chunk
// g = (s / KH)*4 + (s % 32) / 8, element s % 8; the 16-byte chunk (part, g, ch) holds
// channel ch of those 8 keys.  A part thus holds the block rows 32*part .. 32*part+31 and
// KH + 32*part .. KH + 32*part + 31 (the reordering stays inside a 16-key group).
template <int D>
using v_rows = u16[64 * (D + 2)];
template <int D, int BLK, int KEEP>
__device__ __forceinline__ void permute_vtile_part(
    const uint4* __restrict__ v, uint4* __restrict__ vp, const int32_t* __restrict__ perm, int n_blocks, int heads,
    const rf2_strides& st, int block_part, int bh, v_rows<D>& tile) {
  constexpr int CH = D / 8;
  constexpr int RG = 256 / CH;
  constexpr int PITCH = D + 2;       // u16 elements per LDS row: odd number of dwords
  constexpr int PB = BLK / 64, KH = BLK / 2;
  const int blk = block_part / PB, part = block_part % PB;
  const uint4* __restrict__ src = v + ((bh / heads) * st.batch + (bh % heads) * st.head) * CH;
  const int c = threadIdx.x % CH, rg = threadIdx.x / CH;
#pragma unroll
  for (int lr = rg; lr < 64; lr += RG) {                      // local row -> block row
    const int r = (lr / 32) * KH + part * 32 + lr % 32;
    const int n = perm[blk * BLK + r];
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (n >= 0) x = ld_stream<KEEP == 2>(&src[(size_t)n * st.token * CH + c]);
    uint32_t* row = reinterpret_cast<uint32_t*>(tile + lr * PITCH + c * 8);  // 4-byte aligned: PITCH, c*8 even
    row[0] = x.x; row[1] = x.y; row[2] = x.z; row[3] = x.w;
  }
  __syncthreads();
  uint4* __restrict__ dst = vp + (((size_t)bh * n_blocks + blk) * PB + part) * D * 8;
  for (int o = threadIdx.x; o < D * 8; o += 256) {
    const int g = o / D, ch = o % D;   // consecutive lanes -> consecutive channels: contiguous 16-byte stores
    const int sbase = (g / 4) * 32 + (g % 4) * 8;             // first local storage position of this chunk
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int s0 = sbase + 2 * e, s1 = s0 + 1;
      const int k0 = (s0 & ~15) + rho(s0 & 15), k1 = (s1 & ~15) + rho(s1 & 15);
      w[e] = (uint32_t)tile[k0 * PITCH + ch] | ((uint32_t)tile[k1 * PITCH + ch] << 16);
    }
    st_stream<KEEP >= 1>(&dst[o], make_uint4(w[0], w[1], w[2], w[3]));
  }
}

// The three tensors in one launch: first the Q blocks of all heads, then the K blocks, then the V parts.
// Bound by HBM (each byte is read once and written once) where there is enough of it, by the launch elsewhere.  One launch
// against one for each tensor (us): 4,096 tokens x 24 heads 35.9 -> 27.9, x 2 heads 17.4 -> 8.6, 480p x 5 heads 51.9 ->
// 44.8, x 40 344 -> 341 (5.9 TB/s), 720p x 40 784 -> 790; d = 64: 480p x 40 176 -> 168.  With the heads in the outer place
// (Q, K, V of a head in turn) the streams of three tensors are mixed: 30.9, 8.6, 46.4, 342, 796 and 168 us.
struct PermuteArgs {
  const uint4 *q, *k, *v;
  uint4 *qp, *kp, *vp;
  float *qbar, *kbar;
  const int32_t* perm;
  uint32_t n_q, n_k, bh;            // Q and K blocks of a head, heads of all batches
  uint32_t q_wgs, k_wgs, v_wgs;     // workgroups of the launch for each tensor
  int last_q, last_k, heads;
  rf2_strides st;
};
// KEEP: 0 streams past the caches, 1 keeps what it writes, 2 also what it reads.
template <int D, int BQ, int BK, int KEEP>
__global__ void __launch_bounds__(256) permute_kernel(PermuteArgs a) {
  __shared__ __attribute__((aligned(16))) union { pool_rows<D> sums; v_rows<D> tile; } lds;
  uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
  if (id < a.q_wgs) {
    permute_pool_block<D, BQ, false, KEEP>(a.q, a.qp, a.qbar, a.perm, a.n_q, a.last_q, a.heads, a.st, id % a.n_q, id / a.n_q, lds.sums);
    return;
  }
  id -= a.q_wgs;
  if (id < a.k_wgs) {
    permute_pool_block<D, BK, true, KEEP>(a.k, a.kp, a.kbar, a.perm, a.n_k, a.last_k, a.heads, a.st, id % a.n_k, id / a.n_k, lds.sums);
    return;
  }
  id -= a.k_wgs;
  const uint32_t parts = a.n_k * (BK / 64);
  if (id < a.v_wgs) permute_vtile_part<D, BK, KEEP>(a.v, a.vp, a.perm, a.n_k, a.heads, a.st, id % parts, id / parts, lds.tile);
}

// o[n] = op[inv[n]]: gathered reads, fully sequential writes.
template <int D, bool KEEP>
__global__ void __launch_bounds__(256) unpermute_kernel(
    const uint4* __restrict__ op, uint4* __restrict__ o, const int32_t* __restrict__ inv, int N, size_t N_pad,
    int heads, rf2_strides st) {
  constexpr int CH = D / 8;
  constexpr int RG = 256 / CH;
  const int bh = blockIdx.y;
  const uint4* __restrict__ src = op + (size_t)bh * N_pad * CH;
  uint4* __restrict__ dst = o + ((bh / heads) * st.batch + (bh % heads) * st.head) * CH;
  const int c = threadIdx.x % CH, rg = threadIdx.x / CH;
  const int n0 = blockIdx.x * 128;
#pragma unroll 4
  for (int r = rg; r < 128; r += RG) {
    const int n = n0 + r;
    if (n < N) st_stream<false>(&dst[(size_t)n * st.token * CH + c], ld_stream<KEEP>(&src[(size_t)inv[n] * CH + c]));
  }
}

}  // namespace

namespace {

// Whether what is written for one of the three tensors shares memory with what is read or written for another: a caller
// may lay kp over q, and vp over k or q, to save a buffer.
bool tensors_overlap(const rf2_plan* plan, const PermuteArgs& a) {
  const rf2_info& in = plan->info;
  const uint64_t row = (uint64_t)a.bh * plan->cfg.head_dim * 2;
  struct Range { const void* at; uint64_t bytes; int tensor; bool written; };
  const Range r[] = {{a.q, row * in.N, 0, false}, {a.k, row * in.N, 1, false}, {a.v, row * in.N, 2, false},
                     {a.qp, row * in.N_pad, 0, true}, {a.kp, row * in.N_pad_k, 1, true}, {a.vp, row * in.N_pad_k, 2, true},
                     {a.qbar, a.qbar ? row * 2 * a.n_q : 0, 0, true}, {a.kbar, a.kbar ? row * 2 * a.n_k : 0, 1, true}};
  for (const Range& x : r)
    for (const Range& y : r)
      if (x.written && x.tensor != y.tensor && (uint64_t)x.at < (uint64_t)y.at + y.bytes &&
          (uint64_t)y.at < (uint64_t)x.at + x.bytes)
        return true;
  return false;
}

template <int D, int BQ, int BK>
int launch_permute(const rf2_plan* plan, PermuteArgs a, uint32_t q_wgs, uint32_t k_wgs, uint32_t v_wgs, hipStream_t st) {
  // at most (2,048 + 2,048 + 4,096) x 65,535 workgroups, in equal rows of at most 65,536 (a grid dimension holds fewer
  // than 2^32 threads)
  const uint32_t n = q_wgs + k_wgs + v_wgs, rows = (n + 65535u) / 65536u;
  a.q_wgs = q_wgs, a.k_wgs = k_wgs, a.v_wgs = v_wgs;
  const dim3 grid((n + rows - 1) / rows, rows);
  const int64_t bytes = (3 * plan->info.N + plan->info.N_pad + 2 * plan->info.N_pad_k) * (int64_t)a.bh * D * 2;
  if (bytes <= KEEP_ALL) permute_kernel<D, BQ, BK, 2><<<grid, 256, 0, st>>>(a);
  else if (bytes <= KEEP_STORES) permute_kernel<D, BQ, BK, 1><<<grid, 256, 0, st>>>(a);
  else permute_kernel<D, BQ, BK, 0><<<grid, 256, 0, st>>>(a);
  RF2_LAUNCH_CHECK();
  return RF2_OK;
}

template <int D, int BQ, int BK>
int permute_all(const rf2_plan* plan, const PermuteArgs& a, hipStream_t st) {
  const uint32_t q = a.n_q * a.bh, k = a.n_k * a.bh, v = k * (BK / 64);
  if (!tensors_overlap(plan, a)) return launch_permute<D, BQ, BK>(plan, a, q, k, v, st);
  if (const int rc = launch_permute<D, BQ, BK>(plan, a, q, 0, 0, st)) return rc;
  if (const int rc = launch_permute<D, BQ, BK>(plan, a, 0, k, 0, st)) return rc;
  return launch_permute<D, BQ, BK>(plan, a, 0, 0, v, st);
}

template <int D>
int permute_for_dim(const rf2_plan* plan, const PermuteArgs& a, hipStream_t st) {
  const int bq = plan->cfg.block, bk = plan->info.block_k;
#define RF2_PERMUTE_CASE(Q, K) if (bq == Q && bk == K) return permute_all<D, Q, K>(plan, a, st);
  RF2_PERMUTE_CASE(64, 64)
  RF2_PERMUTE_CASE(64, 128)
  RF2_PERMUTE_CASE(128, 64)
  RF2_PERMUTE_CASE(128, 128)
  RF2_PERMUTE_CASE(256, 64)
  RF2_PERMUTE_CASE(256, 128)
#undef RF2_PERMUTE_CASE
  return RF2_ERR_UNSUPPORTED;
}

}  // namespace

extern "C" int rf2_permute(const rf2_plan* plan, const void* q, const void* k, const void* v, void* qp, void* kp,
                           void* vp, float* qbar, float* kbar, void* stream) {
  if (!plan || !q || !k || !v || !qp || !kp || !vp) return RF2_ERR_INVALID_ARG;
  if ((qbar == nullptr) != (kbar == nullptr)) return RF2_ERR_INVALID_ARG;
  if (const int rc = rf2_check_device(plan)) return rc;
  hipStream_t st = (hipStream_t)stream;
  const rf2_info& in = plan->info;
  const PermuteArgs a{(const uint4*)q, (const uint4*)k, (const uint4*)v, (uint4*)qp, (uint4*)kp, (uint4*)vp, qbar, kbar,
                      plan->d_perm, (uint32_t)in.n_blocks, (uint32_t)in.n_blocks_k,
                      (uint32_t)(plan->cfg.batch * plan->cfg.heads), 0, 0, 0, in.last_block_valid, in.last_block_valid_k,
                      plan->cfg.heads, rf2_qkv_strides(plan)};
  if (plan->cfg.head_dim == 128) return permute_for_dim<128>(plan, a, st);
  if (plan->cfg.head_dim == 64) return permute_for_dim<64>(plan, a, st);
  return RF2_ERR_UNSUPPORTED;
}

extern "C" int rf2_unpermute(const rf2_plan* plan, const void* op, void* o, void* stream) {
  if (!plan || !op || !o) return RF2_ERR_INVALID_ARG;
  if (const int rc = rf2_check_device(plan)) return rc;
  const rf2_config& c = plan->cfg;
  const rf2_info& in = plan->info;
  hipStream_t st = (hipStream_t)stream;
  const dim3 grid((unsigned)((in.N + 127) / 128), c.batch * c.heads, 1);
  const bool keep = 2 * in.N * c.batch * c.heads * (int64_t)c.head_dim * 2 <= KEEP_UNPERMUTE;
  const auto launch = [&](auto kernel) {
    kernel<<<grid, 256, 0, st>>>((const uint4*)op, (uint4*)o, plan->d_inv, (int)in.N, (size_t)in.N_pad, c.heads, rf2_qkv_strides(plan));
  };
  if (c.head_dim == 128) keep ? launch(unpermute_kernel<128, true>) : launch(unpermute_kernel<128, false>);
  else keep ? launch(unpermute_kernel<64, true>) : launch(unpermute_kernel<64, false>);
  RF2_LAUNCH_CHECK();
  return RF2_OK;
}
