// The whole message-passing network in a few launches: forward (one of both
// embeddings, two per round) and backward (one of the head, two per round, the
// last with the constraint embedding, two for the weight gradients).  Same
// arithmetic as the single kernels of mpnn.hip: activations and output gradients enter the
// bf16 matrix products as two bf16 parts, weight gradients as three of the four
// cross products; the forward pass is the same operation by operation, so its
// values (and the signs of its activations, which the backward pass masks by)
// are those of the single kernels bit for bit.
//
// Bound by launches and by the latency of the gathers at training size (16
// instances of 200 variables: 840 waves of constraints), by the gathers' and
// rows' bytes at thousands of variables.  A wave takes 16 rows of nodes: the
// dense product of the node's own state (MFMA), the gathered messages, the
// activation and the next product of the new state follow each other in
// registers and a wave's own LDS rows, where the single kernels wrote every
// intermediate and read it back.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "../../include/pcls_mpnn.h"

namespace pcls_mpnn {
int32_t fail(int32_t code, const char* what);
int32_t hip_check(hipError_t e, const char* what);
}  // namespace pcls_mpnn

namespace {

using pcls_mpnn::fail;
using pcls_mpnn::hip_check;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int kHid = 64, kFeat = 32, kLayers = 3;

// ------------------------------------------------------------- parameters
// Offsets (elements) of the flat parameter vector, in the order of the header.
constexpr int kEv = 0, kev = kEv + kHid * kFeat, kEc = kev + kHid, kec = kEc + kHid * kFeat, kLayer0 = kec + kHid;
constexpr int kW1 = 0, kbc = kW1 + kHid * kHid, kWpn = kbc + kHid, kW2 = kWpn + 2 * kHid * kHid,
              kbv = kW2 + kHid * kHid, kUpn = kbv + kHid, kLayerSize = kUpn + 2 * kHid * kHid;
constexpr int kWo = kLayer0 + kLayers * kLayerSize, kBo = kWo + kHid, kParams = kBo + 1;
constexpr int layer_at(int l, int what) { return kLayer0 + l * kLayerSize + what; }

// ------------------------------------------------------------- fragments
// v_mfma_f32_16x16x32_bf16: lane holds A[lane % 16][8 (lane / 16) + e] and
// B[8 (lane / 16) + e][lane % 16], and C[4 (lane / 16) + e][lane % 16].  The
// columns of the product are dealt so that a lane's four 16-column tiles are
// four neighbouring ones: column of tile j, lane l is 4 (l % 16) + j, so C is
// loaded and stored as float4.
struct Split {
  bf16x8 hi, lo;
};

__device__ __forceinline__ Split split8(const float* v) {
  Split s;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = (__bf16)v[e];
    s.hi[e] = h;
    s.lo[e] = (__bf16)(v[e] - (float)h);
  }
  return s;
}
__device__ __forceinline__ Split split8(const float4& a, const float4& b) {
  const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  return split8(v);
}

// op(W) staged in LDS as rows of K (+ 8: the 16 lanes of a tile then start in 16
// different groups of four banks), row h 64 + j 16 + l for column h 64 + 4 l + j.
__device__ __forceinline__ int staged_row(int col) { return (col & ~63) + (col & 3) * 16 + ((col & 63) >> 2); }

// Staging in two halves, so that the loads are in flight while the first rows'
// messages are gathered: eight elements a piece, kPieces of them a thread.
// W stored [COLS][K], or (kT) stored [K][64], transposed on the way into LDS.
template <int COLS, int K, bool kT>
struct Stage {
  static constexpr int kPieces = COLS * K / 8 / 256;
  u32x4 v[kPieces];
  __device__ __forceinline__ void load(const uint16_t* W) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) v[i] = reinterpret_cast<const u32x4*>(W)[i * 256 + threadIdx.x];
  }
  __device__ __forceinline__ void store(__bf16* dst) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int p = i * 256 + threadIdx.x;
      if constexpr (!kT) {
        *reinterpret_cast<u32x4*>(dst + staged_row(p / (K / 8)) * (K + 8) + 8 * (p % (K / 8))) = v[i];
      } else {
        const int k = p / 8, c = 8 * (p % 8);
        uint16_t* d = reinterpret_cast<uint16_t*>(dst);
#pragma unroll
        for (int e = 0; e < 8; ++e) d[staged_row(c + e) * (K + 8) + k] = (uint16_t)(v[i][e / 2] >> (16 * (e & 1)));
      }
    }
  }
};

// acc[j] += A (16 rows, K) times 64 staged columns
template <int K>
__device__ __forceinline__ void product(floatx4 (&acc)[4], const Split (&a)[K / 32], const __bf16* w, int lane) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int k = 0; k < K / 32; ++k) {
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(w + (j * 16 + (lane & 15)) * (K + 8) + 32 * k + 8 * (lane >> 4));
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k].hi, b, acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k].lo, b, acc[j], 0, 0, 0);
    }
  }
}

// the wave's 16 rows as A operand (rows past the end repeat the last one)
template <int K>
__device__ __forceinline__ void load_rows(Split (&a)[K / 32], const float* X, int row0, int N, int lane) {
  const float* p = X + (size_t)min(row0 + (lane & 15), N - 1) * K + 8 * (lane >> 4);
#pragma unroll
  for (int k = 0; k < K / 32; ++k)
    a[k] = split8(*reinterpret_cast<const float4*>(p + 32 * k), *reinterpret_cast<const float4*>(p + 32 * k + 4));
}
template <int K>
__device__ __forceinline__ void load_lds_rows(Split (&a)[K / 32], const float* h, int lane) {
  const float* p = h + (lane & 15) * (K + 4) + 8 * (lane >> 4);
#pragma unroll
  for (int k = 0; k < K / 32; ++k)
    a[k] = split8(*reinterpret_cast<const float4*>(p + 32 * k), *reinterpret_cast<const float4*>(p + 32 * k + 4));
}

__device__ __forceinline__ float relu(float z) { return z > 0.f ? z : 0.f; }

// A wave's own LDS rows are written and read by that wave alone: LDS operations of
// a wave complete in order, only the compiler has to keep the order.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// CSR of one direction: row r has entries ptr[r]..ptr[r+1], idx = (source << 1) | negated.
struct Csr {
  const int32_t* ptr;
  const int32_t* idx;
  const float* w;
};

// Messages of four rows (4 (lane / 16) + e of the wave's 16) at columns
// 4 (lane % 16)..+3.  kSplit false: In has both sign halves side by side, one sum a
// row; true: In has 64 columns, one sum per sign.  Entries of a row are added in
// order.  The 16 lanes of a row group load 16 entries at once and pass them round,
// so only the rows of In are waited for: four rows times four entries in flight
// (with every entry's index loaded before its row, two entries deep, a round of
// 3200 variables of degree 12.6 took 25 us).
template <bool kSplit>
__device__ __forceinline__ void gather4(const Csr& g, const float* In, int row0, int N, int lane, float4 (&p)[4],
                                        float4 (&n)[4]) {
  int at[4], len[4], most = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = row0 + 4 * (lane >> 4) + e;
    at[e] = r < N ? g.ptr[r] : 0;
    len[e] = r < N ? g.ptr[r + 1] - at[e] : 0;
    p[e] = n[e] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) most = max(most, len[e]);
  most = max(most, __shfl_xor(most, 16));
  most = max(most, __shfl_xor(most, 32));  // of the whole wave: the exchanges below need every lane
  const int c4 = 4 * (lane & 15), l = lane & 15, group = lane & 48;
  constexpr int kDeep = 4;
  for (int j0 = 0; j0 < most; j0 += 16) {
    int code[4];
    float w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      code[e] = 0;
      w[e] = 0.f;
      if (j0 + l < len[e]) {
        code[e] = g.idx[at[e] + j0 + l];
        w[e] = g.w[at[e] + j0 + l];
      }
    }
    const int stop = min(most - j0, 16);
    for (int j = 0; j < stop; j += kDeep) {
      float4 x[4][kDeep];
      int cj[4][kDeep];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
          cj[e][d] = __shfl(code[e], group + j + d);
          if (j0 + j + d < len[e])
            x[e][d] = *reinterpret_cast<const float4*>(
                In + (size_t)(cj[e][d] >> 1) * (kSplit ? 64 : 128) + (kSplit ? 0 : 64 * (cj[e][d] & 1)) + c4);
        }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
          const float wj = __shfl(w[e], group + j + d);
          if (j0 + j + d < len[e]) {
            float4& s = kSplit && (cj[e][d] & 1) ? n[e] : p[e];
            s.x = fmaf(wj, x[e][d].x, s.x);
            s.y = fmaf(wj, x[e][d].y, s.y);
            s.z = fmaf(wj, x[e][d].z, s.z);
            s.w = fmaf(wj, x[e][d].w, s.w);
          }
        }
    }
  }
}

// Few nodes: 16 rows a wave leave CUs idle, and a row's entries come in latencies of
// four.  There the block's four waves gather for the same 16 rows, one row a lane group
// with 16 entries in flight, and the first goes on with the messages from LDS.
// Measured for one side against 16 rows a wave (forward pass and training step, us;
// n x k: n rows of about k entries):
//   800 x 12.6    79 -> 52, 185 -> 133    8192 x 3    70 -> 59, 166 -> 143
//   3200 x 12.6   96 -> 69, 218 -> 164    8000 x 5    83 -> 64, 187 -> 150
//   10000 x 3     77 -> 75, 176 -> 185    12000 x 3   78 -> 82, 193 -> 206
//   10000 x 6     93 -> 83, 222 -> 212    12000 x 9  116 -> 105, 298 -> 288
//   16000 x 5     92 -> 93, 227 -> 237    16000 x 6   96 -> 94, 255 -> 257
//   16000 x 12.6 157 -> 148, 451 -> 450   24000 x 12.6 188 -> 195, 592 -> 626
// Up to kSharedRows, 512 blocks, two a CU (all that back_kernel's LDS lets a CU hold),
// it is faster at any length; up to twice as many only for long rows.  The host does
// not know the lengths: it takes variables with at least two constraints each, whose
// rows are long where constraints are of three literals or more.
constexpr int kSharedRows = 8192;

// Messages of one row, 4 (lane / 16) + e of the 16; as gather4 otherwise
template <bool kSplit>
__device__ __forceinline__ void gather1(const Csr& g, const float* In, int row0, int N, int lane, int e, float4& p,
                                        float4& n) {
  const int r = row0 + 4 * (lane >> 4) + e;
  const int at = r < N ? g.ptr[r] : 0, len = r < N ? g.ptr[r + 1] - at : 0;
  int most = max(len, __shfl_xor(len, 16));
  most = max(most, __shfl_xor(most, 32));
  const int c4 = 4 * (lane & 15), l = lane & 15, group = lane & 48;
  p = n = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int j0 = 0; j0 < most; j0 += 16) {
    int code = 0;
    float w = 0.f;
    if (j0 + l < len) {
      code = g.idx[at + j0 + l];
      w = g.w[at + j0 + l];
    }
    float4 x[16];
    int cj[16];
#pragma unroll
    for (int d = 0; d < 16; ++d) {
      cj[d] = __shfl(code, group + d);
      if (j0 + d < len)
        x[d] = *reinterpret_cast<const float4*>(In + (size_t)(cj[d] >> 1) * (kSplit ? 64 : 128) +
                                                (kSplit ? 0 : 64 * (cj[d] & 1)) + c4);
    }
#pragma unroll
    for (int d = 0; d < 16; ++d) {
      const float wj = __shfl(w, group + d);
      if (j0 + d < len) {
        float4& s = kSplit && (cj[d] & 1) ? n : p;
        s.x = fmaf(wj, x[d].x, s.x);
        s.y = fmaf(wj, x[d].y, s.y);
        s.z = fmaf(wj, x[d].z, s.z);
        s.w = fmaf(wj, x[d].w, s.w);
      }
    }
  }
}

// ---------------------------------------------------------------- forward
// H = relu(F E^T + e); P = H Wn^T (128 columns)
struct EmbedArgs {
  const float* F;
  int N;
  const uint16_t* E;
  const float* e;
  float* H;
  const uint16_t* Wn;  // [128][64] or NULL
  float* P;
};

// Two sides that do not wait for each other share a launch: the first blocks0
// blocks take V, the rest C (embedding and last backward launch: a launch of few
// blocks costs its latency whatever it does: predict 8 x 2000 variables 151 -> 149 us,
// training 16 x 200 222 -> 213 us, with the two-step meeting of wgrad_kernel's waves).
__global__ void __launch_bounds__(256) embed_kernel(EmbedArgs V, int blocks0, EmbedArgs C) {
  const bool second = (int)blockIdx.x >= blocks0;
  const EmbedArgs A = second ? C : V;
  const int block = blockIdx.x - (second ? blocks0 : 0), blocks = second ? gridDim.x - blocks0 : blocks0;
  __shared__ __attribute__((aligned(16))) __bf16 we[64 * (kFeat + 8)], wn[128 * (kHid + 8)];
  __shared__ __attribute__((aligned(16))) float hs[4][16 * (kHid + 4)];
  Stage<64, kFeat, false> se;
  Stage<128, kHid, false> sn;
  se.load(A.E);
  if (A.Wn) sn.load(A.Wn);
  se.store(we);
  if (A.Wn) sn.store(wn);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c4 = 4 * (lane & 15);
  const float4 b = *reinterpret_cast<const float4*>(A.e + c4);
  for (int row0 = (block * 4 + wave) * 16; row0 < A.N; row0 += blocks * 64) {
    Split f[1];
    load_rows<kFeat>(f, A.F, row0, A.N, lane);
    floatx4 acc[4] = {};
    product<kFeat>(acc, f, we, lane);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * (lane >> 4) + e;
      const float4 h = make_float4(relu(acc[0][e] + b.x), relu(acc[1][e] + b.y), relu(acc[2][e] + b.z), relu(acc[3][e] + b.w));
      if (row0 + r < A.N) *reinterpret_cast<float4*>(A.H + (size_t)(row0 + r) * 64 + c4) = h;
      *reinterpret_cast<float4*>(&hs[wave][r * (kHid + 4) + c4]) = h;
    }
    if (!A.Wn) continue;
    wave_order();
    Split a[2];
    load_lds_rows<kHid>(a, hs[wave], lane);
    wave_order();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      floatx4 q[4] = {};
      product<kHid>(q, a, wn + h * 64 * (kHid + 8), lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = row0 + 4 * (lane >> 4) + e;
        if (r < A.N) *reinterpret_cast<float4*>(A.P + (size_t)r * 128 + 64 * h + c4) = make_float4(q[0][e], q[1][e], q[2][e], q[3][e]);
      }
    }
  }
}

// H' = relu((H W^T + b) + messages); then the 128-column product P = H' Wn^T for
// the other side's next gather, or (variables, last round) the output head.
struct RoundArgs {
  const float* H;
  int N;
  const uint16_t* W;
  const float* b;
  Csr g;
  const float* In;
  float* Hout;
  const uint16_t* Wn;  // or NULL
  float* P;
  const float* wo;     // or NULL: xhat = tanh(H' . wo + bo)
  const float* bo;
  float* xhat;
  bool shared;         // gathered by the block together (gather1)
};

__global__ void __launch_bounds__(256) round_kernel(RoundArgs A) {
  __shared__ __attribute__((aligned(16))) __bf16 ws[64 * (kHid + 8)], wn[128 * (kHid + 8)];
  __shared__ __attribute__((aligned(16))) float hs[4][16 * (kHid + 4)];
  Stage<64, kHid, false> sw;
  Stage<128, kHid, false> sn;
  sw.load(A.W);
  if (A.Wn) sn.load(A.Wn);
  bool staged = false;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c4 = 4 * (lane & 15);
  const float4 b = *reinterpret_cast<const float4*>(A.b + c4);
  const bool shared = A.shared;  // one pass of the loop
  for (int row0 = shared ? blockIdx.x * 16 : (blockIdx.x * 4 + wave) * 16;; row0 += gridDim.x * 64) {
    float4 msg[4], none[4];
    if (shared && row0 < A.N) {
      gather1<false>(A.g, A.In, row0, A.N, lane, wave, msg[0], none[0]);
      *reinterpret_cast<float4*>(&hs[1][(4 * (lane >> 4) + wave) * (kHid + 4) + c4]) = msg[0];
    } else if (row0 < A.N) {
      gather4<false>(A.g, A.In, row0, A.N, lane, msg, none);
    }
    if (!staged) {  // every wave comes here once
      sw.store(ws);
      if (A.Wn) sn.store(wn);
      __syncthreads();
      staged = true;
    }
    if (row0 >= A.N) break;
    if (shared) {
      if (wave > 0) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        msg[e] = *reinterpret_cast<const float4*>(&hs[1][(4 * (lane >> 4) + e) * (kHid + 4) + c4]);
    }
    Split a[2];
    load_rows<kHid>(a, A.H, row0, A.N, lane);
    floatx4 acc[4] = {};
    product<kHid>(acc, a, ws, lane);
    float s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * (lane >> 4) + e;
      const float4 h = make_float4(relu((acc[0][e] + b.x) + msg[e].x), relu((acc[1][e] + b.y) + msg[e].y),
                                   relu((acc[2][e] + b.z) + msg[e].z), relu((acc[3][e] + b.w) + msg[e].w));
      if (row0 + r < A.N) *reinterpret_cast<float4*>(A.Hout + (size_t)(row0 + r) * 64 + c4) = h;
      if (A.Wn) *reinterpret_cast<float4*>(&hs[wave][r * (kHid + 4) + c4]) = h;
      if (A.wo) {
        // the sum over 64 columns as the single head kernel forms it: columns 32
        // apart first (one rounded product, one fused), then 16, 8, 4, 2, 1
        const float4 w = *reinterpret_cast<const float4*>(A.wo + c4);
        float t[4] = {__fmul_rn(h.x, w.x), __fmul_rn(h.y, w.y), __fmul_rn(h.z, w.z), __fmul_rn(h.w, w.w)};
        const float hv[4] = {h.x, h.y, h.z, h.w}, wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = fmaf(hv[j], wv[j], __shfl_xor(t[j], 8));
#pragma unroll
        for (int o = 4; o > 0; o >>= 1)
#pragma unroll
          for (int j = 0; j < 4; ++j) t[j] += __shfl_xor(t[j], o);
        s[e] = (t[0] + t[2]) + (t[1] + t[3]);
      }
    }
    if (A.wo) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = row0 + 4 * (lane >> 4) + e;
        if ((lane & 15) == 0 && r < A.N) A.xhat[r] = tanhf(s[e] + A.bo[0]);
      }
    }
    if (!A.Wn) continue;
    wave_order();
    load_lds_rows<kHid>(a, hs[wave], lane);
    wave_order();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      floatx4 q[4] = {};
      product<kHid>(q, a, wn + h * 64 * (kHid + 8), lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = row0 + 4 * (lane >> 4) + e;
        if (r < A.N) *reinterpret_cast<float4*>(A.P + (size_t)r * 128 + 64 * h + c4) = make_float4(q[0][e], q[1][e], q[2][e], q[3][e]);
      }
    }
  }
}

// --------------------------------------------------------------- backward
// dlogit = dxhat (1 - xhat^2); dZ = dlogit wo where the activation was positive
__global__ void head_back_kernel(const float* __restrict__ xhat, const float* __restrict__ dxhat, int N,
                                 const float* __restrict__ wo, const float* __restrict__ H, float* __restrict__ dZ,
                                 float* __restrict__ dlogit) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = i >> 4, c4 = 4 * (i & 15);
  if (r >= N) return;
  const float x = xhat[r], d = dxhat[r] * (1.f - x * x);
  const float4 w = *reinterpret_cast<const float4*>(wo + c4), h = *reinterpret_cast<const float4*>(H + (size_t)r * 64 + c4);
  *reinterpret_cast<float4*>(dZ + (size_t)r * 64 + c4) =
      make_float4(h.x > 0.f ? d * w.x : 0.f, h.y > 0.f ? d * w.y : 0.f, h.z > 0.f ? d * w.z : 0.f, h.w > 0.f ? d * w.w : 0.f);
  if (c4 == 0) dlogit[r] = d;
}

// dQ = the gathered output gradients by sign (128 columns); dZ = (dQ Wbig +
// dSelf Wself) where the activation H was positive.
struct BackArgs {
  int N;
  Csr g;
  const float* In;       // [sources][64], or NULL: no gather
  const uint16_t* Wbig;  // [128][64]
  float* dQ;             // [N][128]
  const float* dSelf;    // [N][64] or NULL
  const uint16_t* Wself; // [64][64]
  const float* H;        // [N][64]
  float* dZ;             // [N][64]
  bool shared;           // gathered by the block together (gather1)
};

// blocks0 as in embed_kernel
__global__ void __launch_bounds__(256) back_kernel(BackArgs V, int blocks0, BackArgs C) {
  const bool second = (int)blockIdx.x >= blocks0;
  const BackArgs A = second ? C : V;
  const int block = blockIdx.x - (second ? blocks0 : 0), blocks = second ? gridDim.x - blocks0 : blocks0;
  __shared__ __attribute__((aligned(16))) __bf16 wb[64 * (128 + 8)], ws[64 * (kHid + 8)];
  __shared__ __attribute__((aligned(16))) float qs[4][16 * (128 + 4)];
  Stage<64, 128, true> sb;
  Stage<64, kHid, true> sw;
  if (A.In) sb.load(A.Wbig);
  if (A.dSelf) sw.load(A.Wself);
  bool staged = false;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c4 = 4 * (lane & 15);
  const bool shared = A.shared;  // one pass of the loop
  for (int row0 = shared ? block * 16 : (block * 4 + wave) * 16;; row0 += blocks * 64) {
    floatx4 acc[4] = {};
    float4 p[4], n[4];
    if (shared && row0 < A.N) {
      gather1<true>(A.g, A.In, row0, A.N, lane, wave, p[0], n[0]);
      const int r = 4 * (lane >> 4) + wave;
      if (row0 + r < A.N) {
        *reinterpret_cast<float4*>(A.dQ + (size_t)(row0 + r) * 128 + c4) = p[0];
        *reinterpret_cast<float4*>(A.dQ + (size_t)(row0 + r) * 128 + 64 + c4) = n[0];
      }
      *reinterpret_cast<float4*>(&qs[0][r * 132 + c4]) = p[0];
      *reinterpret_cast<float4*>(&qs[0][r * 132 + 64 + c4]) = n[0];
    } else if (A.In && row0 < A.N) {
      gather4<true>(A.g, A.In, row0, A.N, lane, p, n);
    }
    if (!staged) {  // every wave comes here once
      if (A.In) sb.store(wb);
      if (A.dSelf) sw.store(ws);
      __syncthreads();
      staged = true;
    }
    if (row0 >= A.N || (shared && wave > 0)) break;
    if (A.In) {
      if (!shared) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * (lane >> 4) + e;
          if (row0 + r < A.N) {
            *reinterpret_cast<float4*>(A.dQ + (size_t)(row0 + r) * 128 + c4) = p[e];
            *reinterpret_cast<float4*>(A.dQ + (size_t)(row0 + r) * 128 + 64 + c4) = n[e];
          }
          *reinterpret_cast<float4*>(&qs[wave][r * 132 + c4]) = p[e];
          *reinterpret_cast<float4*>(&qs[wave][r * 132 + 64 + c4]) = n[e];
        }
      }
      wave_order();
      Split a[4];
      load_lds_rows<128>(a, qs[wave], lane);
      wave_order();
      product<128>(acc, a, wb, lane);
    }
    if (A.dSelf) {
      Split a[2];
      load_rows<kHid>(a, A.dSelf, row0, A.N, lane);
      product<kHid>(acc, a, ws, lane);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = row0 + 4 * (lane >> 4) + e;
      if (r >= A.N) continue;
      const float4 h = *reinterpret_cast<const float4*>(A.H + (size_t)r * 64 + c4);
      *reinterpret_cast<float4*>(A.dZ + (size_t)r * 64 + c4) =
          make_float4(h.x > 0.f ? acc[0][e] : 0.f, h.y > 0.f ? acc[1][e] : 0.f, h.z > 0.f ? acc[2][e] : 0.f,
                      h.w > 0.f ? acc[3][e] : 0.f);
    }
  }
}

// Every weight gradient in one launch: dW[64][K] = sum_n dZ[n][.]^T X[n][.] over 64
// columns of dZ (128-column gradients are two of these), the bias gradient its
// column sums.  A block takes a chunk of rows of one product, a wave 32 rows at a
// time with all of the product's tiles: one float4 per row and lane serves the
// four tiles (column of tile j: 4 (lane % 16) + j), so every element is read and
// split once.  The waves' sums meet in LDS, the chunks' in wgrad_sum_kernel, both
// in a fixed order.
constexpr int kMaxGrads = 3 * 6 + 3;
struct Grad {
  const float* dZ;    // [N][ldz], 64 columns used
  const float* X;     // [N][K]; K = 1: the head (dZ has one column, X 64)
  int ldz, K, N;
  int out, bias;      // offsets into the gradient; bias < 0: none
  int block0, chunks; // first block, blocks
  int part;           // offset of the first chunk's partial sums (floats)
};
struct Grads {
  Grad g[kMaxGrads];
  int count, rows;    // rows of a chunk (a multiple of 128)
};
constexpr int partial_size(int K) { return K == 1 ? 128 : 64 * K + 64; }

template <int K>
__device__ __forceinline__ void grad_chunk(const Grad& G, int begin, int end, float* out, float* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c4 = 4 * (lane & 15), rq = 8 * (lane >> 4);
  constexpr int KT = K / 16;  // tiles of X; K = 32: column of tile j is 2 (lane % 16) + j
  floatx4 acc[4][KT] = {};
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int n0 = begin + 32 * wave; n0 < end; n0 += 128) {
    float z[4][8], x[KT][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int n = n0 + rq + e;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f), y = v;
      if (n < end) {
        v = *reinterpret_cast<const float4*>(G.dZ + (size_t)n * G.ldz + c4);
        if constexpr (K == 64) {
          y = *reinterpret_cast<const float4*>(G.X + (size_t)n * K + c4);
        } else {
          const float2 t = *reinterpret_cast<const float2*>(G.X + (size_t)n * K + (c4 >> 1));
          y.x = t.x;
          y.y = t.y;
        }
      }
      sum.x += v.x;
      sum.y += v.y;
      sum.z += v.z;
      sum.w += v.w;
      z[0][e] = v.x;
      z[1][e] = v.y;
      z[2][e] = v.z;
      z[3][e] = v.w;
      x[0][e] = y.x;
      x[1][e] = y.y;
      if constexpr (KT == 4) {
        x[2][e] = y.z;
        x[3][e] = y.w;
      }
    }
    Split b[KT];
#pragma unroll
    for (int j = 0; j < KT; ++j) b[j] = split8(x[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const Split a = split8(z[i]);
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b[j].hi, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b[j].lo, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.lo, b[j].hi, acc[i][j], 0, 0, 0);
      }
    }
  }
  // column sums over the four groups of rows
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    sum.x += __shfl_xor(sum.x, o);
    sum.y += __shfl_xor(sum.y, o);
    sum.z += __shfl_xor(sum.z, o);
    sum.w += __shfl_xor(sum.w, o);
  }
  // waves 0 and 1 store their tiles, 2 and 3 add theirs, the store to memory adds the
  // two; element (m, k), m = 4 (row of the tile) + i, k = KT (lane % 16) + j
  float* half = lds + (wave & 1) * (64 * 64 + 64);
  for (int w = 0; w < 2; ++w) {
    if (wave >> 1 == w) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float* p = half + (size_t)(4 * (4 * (lane >> 4) + e) + i) * K + KT * (lane & 15);
#pragma unroll
          for (int j = 0; j < KT; ++j) p[j] = w == 0 ? acc[i][j][e] : p[j] + acc[i][j][e];
        }
      if (lane < 16) {
        float* p = half + 64 * K + c4;
        p[0] = w == 0 ? sum.x : p[0] + sum.x;
        p[1] = w == 0 ? sum.y : p[1] + sum.y;
        p[2] = w == 0 ? sum.z : p[2] + sum.z;
        p[3] = w == 0 ? sum.w : p[3] + sum.w;
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < 64 * K + 64; i += blockDim.x) out[i] = lds[i] + lds[64 * 64 + 64 + i];
}

__global__ void __launch_bounds__(256) wgrad_kernel(Grads A, float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) float lds[2 * (64 * 64 + 64)];
  int q = 0;
  while (q + 1 < A.count && (int)blockIdx.x >= A.g[q + 1].block0) ++q;
  const Grad G = A.g[q];
  const int chunk = blockIdx.x - G.block0;
  const int begin = chunk * A.rows, end = min(G.N, begin + A.rows);
  float* out = partial + G.part + (size_t)chunk * partial_size(G.K);
  if (G.K == 64) {
    grad_chunk<64>(G, begin, end, out, lds);
  } else if (G.K == 32) {
    grad_chunk<32>(G, begin, end, out, lds);
  } else {  // head: out[d] = sum_n dlogit[n] H[n][d], out[64] = sum_n dlogit[n]
    const int d = threadIdx.x & 63, w = threadIdx.x >> 6;
    float s = 0.f, sb = 0.f;
    for (int n = begin + w; n < end; n += 4) {
      const float g = G.dZ[n];
      s = fmaf(g, G.X[(size_t)n * 64 + d], s);
      sb += g;
    }
    lds[w * 64 + d] = s;
    if (d == 0) lds[256 + w] = sb;
    __syncthreads();
    if (w == 0) out[d] = lds[d] + lds[64 + d] + lds[128 + d] + lds[192 + d];
    if (threadIdx.x == 64) out[64] = lds[256] + lds[257] + lds[258] + lds[259];
  }
}

// grad[i] = sum over the chunks' partial sums; blockIdx.y = product
__global__ void __launch_bounds__(256) wgrad_sum_kernel(Grads A, const float* __restrict__ partial,
                                                        float* __restrict__ grad) {
  const Grad G = A.g[blockIdx.y];
  const int size = partial_size(G.K), i = blockIdx.x * blockDim.x + threadIdx.x;
  const int outs = G.K == 1 ? 64 : 64 * G.K, used = G.bias < 0 ? outs : outs + (G.K == 1 ? 1 : 64);
  if (i >= used) return;
  const float* p = partial + G.part + i;
  float s = 0.f;
#pragma unroll 8
  for (int c = 0; c < G.chunks; ++c) s += p[(size_t)c * size];
  grad[i < outs ? G.out + i : G.bias + (i - outs)] = s;
}

// ------------------------------------------------------------------- host
int blocks_for(int N) { return N > 0 ? ((N + 63) / 64 < 1024 ? (N + 63) / 64 : 1024) : 0; }
bool constraints_shared(int Nc) { return Nc <= kSharedRows; }
bool variables_shared(int Nv, int Nc) { return Nv <= kSharedRows || (Nv <= 2 * kSharedRows && 2 * Nv <= Nc); }
// blocks of a kernel that gathers for N rows
int gather_blocks(int N, bool shared) { return shared ? (N + 15) / 16 : blocks_for(N); }

// Activations kept by the forward pass (floats): H of the embedding and of each
// round, variables then constraints, and the two 128-column products.
struct Acts {
  size_t hv[kLayers + 1], hc[kLayers + 1], pm, qm, total;
};
Acts acts_of(size_t Nv, size_t Nc) {
  Acts a;
  size_t at = 0;
  for (int l = 0; l <= kLayers; ++l) {
    a.hv[l] = at;
    at += Nv * kHid;
    a.hc[l] = at;
    at += Nc * kHid;
  }
  a.pm = at;
  at += Nv * 2 * kHid;
  a.qm = at;
  a.total = at + Nc * 2 * kHid;
  return a;
}

// Scratch of the backward pass (floats): gradients before the activations of
// every round, the gathered gradients, dlogit, the weight gradients' partial sums.
struct Back {
  size_t dzv[kLayers + 1], dzc[kLayers + 1], dp[kLayers], dq[kLayers], dlogit, part, total;
  int rows, blocks;
};
int chunks_of(int N, int rows) { return (N + rows - 1) / rows; }
Back back_of(int Nv, int Nc) {
  Back b;
  size_t at = 0;
  const size_t nv = (size_t)Nv, nc = (size_t)Nc;
  for (int l = 0; l <= kLayers; ++l) {
    b.dzv[l] = at;
    at += nv * kHid;
    b.dzc[l] = at;
    at += nc * kHid;
  }
  for (int l = 0; l < kLayers; ++l) {
    b.dp[l] = at;
    at += nv * 2 * kHid;
    b.dq[l] = at;
    at += nc * 2 * kHid;
  }
  b.dlogit = at;
  at += (nv + 63) / 64 * 64;
  b.part = at;
  // chunks of 256 rows: 462 blocks at 3200 variables and 13440 constraints; longer
  // ones where that would be far more blocks than the card holds at once
  const int per = 3 * (3 * chunks_of(Nv, 256) + 3 * chunks_of(Nc, 256));
  b.rows = 256 * (1 + per / 2048);
  const size_t cv = (size_t)chunks_of(Nv, b.rows), cc = (size_t)chunks_of(Nc, b.rows);
  at += (cv + cc) * (3 * 3 * (size_t)partial_size(64) + partial_size(32)) + cv * partial_size(1);
  b.total = at;
  return b;
}

bool bad_graph(const pcls_mpnn_graph* g) {
  return !g || g->n_vars < 0 || g->n_cons < 0 || (g->n_vars > 0 && (!g->feat_v || !g->vptr)) ||
         (g->n_cons > 0 && (!g->feat_c || !g->cptr));
}

}  // namespace

extern "C" {

size_t pcls_mpnn_forward_floats(int32_t n_vars, int32_t n_cons) {
  return n_vars < 0 || n_cons < 0 ? 0 : acts_of((size_t)n_vars, (size_t)n_cons).total;
}

size_t pcls_mpnn_backward_floats(int32_t n_vars, int32_t n_cons) {
  return n_vars < 0 || n_cons < 0 ? 0 : back_of(n_vars, n_cons).total;
}

int32_t pcls_mpnn_forward(const pcls_mpnn_graph* g, const float* params, const uint16_t* params_bf16, float* acts,
                          float* xhat, void* stream) {
  if (bad_graph(g) || !params || !params_bf16 || !acts || (g->n_vars > 0 && !xhat))
    return fail(1, "forward: NULL pointer or negative size");
  if (((uintptr_t)params_bf16 | (uintptr_t)params | (uintptr_t)acts | (uintptr_t)g->feat_v | (uintptr_t)g->feat_c) & 15u)
    return fail(1, "forward: parameters, features and activations must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int Nv = g->n_vars, Nc = g->n_cons;
  const bool cons = constraints_shared(Nc), vars = variables_shared(Nv, Nc);
  const Acts a = acts_of((size_t)Nv, (size_t)Nc);
  if (Nv > 0 || Nc > 0) {
    const EmbedArgs V{g->feat_v,       Nv, params_bf16 + kEv, params + kev, acts + a.hv[0], params_bf16 + layer_at(0, kWpn),
                      acts + a.pm};
    const EmbedArgs C{g->feat_c, Nc, params_bf16 + kEc, params + kec, acts + a.hc[0], nullptr, nullptr};
    hipLaunchKernelGGL(embed_kernel, dim3(blocks_for(Nv) + blocks_for(Nc)), dim3(256), 0, s, V, blocks_for(Nv), C);
  }
  for (int l = 0; l < kLayers; ++l) {
    const bool last = l + 1 == kLayers;
    if (Nc > 0) {
      const RoundArgs C{acts + a.hc[l], Nc, params_bf16 + layer_at(l, kW1), params + layer_at(l, kbc),
                        Csr{g->cptr, g->cidx, g->cw}, acts + a.pm, acts + a.hc[l + 1],
                        params_bf16 + layer_at(l, kUpn), acts + a.qm, nullptr, nullptr, nullptr, cons};
      hipLaunchKernelGGL(round_kernel, dim3(gather_blocks(Nc, cons)), dim3(256), 0, s, C);
    }
    if (Nv > 0) {
      const RoundArgs V{acts + a.hv[l], Nv, params_bf16 + layer_at(l, kW2), params + layer_at(l, kbv),
                        Csr{g->vptr, g->vidx, g->vw}, acts + a.qm, acts + a.hv[l + 1],
                        last ? nullptr : params_bf16 + layer_at(l + 1, kWpn), acts + a.pm,
                        last ? params + kWo : nullptr, params + kBo, xhat, vars};
      hipLaunchKernelGGL(round_kernel, dim3(gather_blocks(Nv, vars)), dim3(256), 0, s, V);
    }
  }
  return hip_check(hipGetLastError(), "forward launch");
}

int32_t pcls_mpnn_backward(const pcls_mpnn_graph* g, const float* params, const uint16_t* params_bf16,
                           const float* acts, const float* xhat, const float* dxhat, float* grad, float* scratch,
                           size_t scratch_floats, void* stream) {
  if (bad_graph(g) || !params || !params_bf16 || !acts || !grad || !scratch || (g->n_vars > 0 && (!xhat || !dxhat)))
    return fail(1, "backward: NULL pointer or negative size");
  if (((uintptr_t)params_bf16 | (uintptr_t)params | (uintptr_t)acts | (uintptr_t)scratch | (uintptr_t)g->feat_v |
       (uintptr_t)g->feat_c) & 15u)
    return fail(1, "backward: parameters, features, activations and scratch must be 16-byte aligned");
  const int Nv = g->n_vars, Nc = g->n_cons;
  const bool cons = constraints_shared(Nc), vars = variables_shared(Nv, Nc);
  const Acts a = acts_of((size_t)Nv, (size_t)Nc);
  const Back b = back_of(Nv, Nc);
  if (scratch_floats < b.total) return fail(4, "backward: scratch too small");
  hipStream_t s = (hipStream_t)stream;
  if (Nv > 0)
    hipLaunchKernelGGL(head_back_kernel, dim3((Nv * 16 + 255) / 256), dim3(256), 0, s, xhat, dxhat, Nv, params + kWo,
                       acts + a.hv[kLayers], scratch + b.dzv[kLayers], scratch + b.dlogit);
  for (int l = kLayers - 1; l >= 0; --l) {
    // index l + 1: gradients before round l's activations; 0: before the embedding's
    if (Nc > 0) {
      const bool top = l + 1 == kLayers;
      const BackArgs C{Nc, Csr{g->cptr, g->cidx, g->cw_t}, scratch + b.dzv[l + 1], params_bf16 + layer_at(l, kUpn),
                       scratch + b.dq[l], top ? nullptr : scratch + b.dzc[l + 2],
                       top ? nullptr : params_bf16 + layer_at(l + 1, kW1), acts + a.hc[l + 1], scratch + b.dzc[l + 1],
                       cons};
      hipLaunchKernelGGL(back_kernel, dim3(gather_blocks(Nc, cons)), dim3(256), 0, s, C, gather_blocks(Nc, cons), C);
    }
    if (Nv > 0 || (l == 0 && Nc > 0)) {
      const BackArgs V{Nv, Csr{g->vptr, g->vidx, g->vw_t}, scratch + b.dzc[l + 1], params_bf16 + layer_at(l, kWpn),
                       scratch + b.dp[l], scratch + b.dzv[l + 1], params_bf16 + layer_at(l, kW2), acts + a.hv[l],
                       scratch + b.dzv[l], vars};
      // the constraint embedding's gradient needs no more than round 0's
      const BackArgs C{Nc, Csr{nullptr, nullptr, nullptr}, nullptr, nullptr, nullptr, scratch + b.dzc[1],
                       params_bf16 + layer_at(0, kW1), acts + a.hc[0], scratch + b.dzc[0], false};
      const int with = l == 0 ? blocks_for(Nc) : 0;
      hipLaunchKernelGGL(back_kernel, dim3(gather_blocks(Nv, vars) + with), dim3(256), 0, s, V, gather_blocks(Nv, vars), C);
    }
  }
  Grads G{};
  G.rows = b.rows;
  int block = 0;
  size_t part = b.part;
  auto add = [&](const float* dZ, int ldz, const float* X, int K, int N, int out, int bias) {
    Grad& q = G.g[G.count++];
    q = Grad{dZ, X, ldz, K, N, out, bias, block, chunks_of(N, b.rows), (int)(part - b.part)};
    block += q.chunks;
    part += (size_t)q.chunks * partial_size(K);
  };
  for (int l = 0; l < kLayers; ++l) {
    const int half = kHid * kHid;
    add(scratch + b.dzv[l + 1], 64, acts + a.hv[l], 64, Nv, layer_at(l, kW2), layer_at(l, kbv));
    add(scratch + b.dzc[l + 1], 64, acts + a.hc[l], 64, Nc, layer_at(l, kW1), layer_at(l, kbc));
    add(scratch + b.dq[l], 128, acts + a.hc[l + 1], 64, Nc, layer_at(l, kUpn), -1);
    add(scratch + b.dq[l] + 64, 128, acts + a.hc[l + 1], 64, Nc, layer_at(l, kUpn) + half, -1);
    add(scratch + b.dp[l], 128, acts + a.hv[l], 64, Nv, layer_at(l, kWpn), -1);
    add(scratch + b.dp[l] + 64, 128, acts + a.hv[l], 64, Nv, layer_at(l, kWpn) + half, -1);
  }
  add(scratch + b.dzv[0], 64, g->feat_v, 32, Nv, kEv, kev);
  add(scratch + b.dzc[0], 64, g->feat_c, 32, Nc, kEc, kec);
  add(scratch + b.dlogit, 1, acts + a.hv[kLayers], 1, Nv, kWo, kBo);
  if (block > 0) hipLaunchKernelGGL(wgrad_kernel, dim3(block), dim3(256), 0, s, G, scratch + b.part);
  hipLaunchKernelGGL(wgrad_sum_kernel, dim3((partial_size(64) + 255) / 256, G.count), dim3(256), 0, s, G,
                     scratch + b.part, grad);
  return hip_check(hipGetLastError(), "backward launch");
}

}  // extern "C"
