// The stacked XOR layers (Eq. 8): rows streamed past stationary weight slices, the products chained through LDS.
#include "mfma.hpp"

namespace lime {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The gated block of an XOR layer (Eq. 8) in one pass over the rows:  Y = X + (A * SiLU(X W_U)) W_O.
// One wave per head-sized slice of the d output columns, both weight slices stationary (A operands).  Per tile of
// 32 rows: P^T = W_U^T X^T from the rows' fragments, the gate on the accumulators (a lane owns one row), the gated
// rows Z through LDS (every wave needs all d columns of Z as the B operand of the second product), Y^T = W_O^T Z^T,
// then the residual and, for link rows, the running fp32 sum of the layers' outputs.
struct GatedArgs {
  const bf16_t* X;        // [.][rows][d] the layer's input rows (gate input and residual)
  int64_t x_user_stride;  // elements between users (0 = shared rows)
  const int32_t* lens;    // nullable; rows >= lens[b] count as zeros and are written as zeros
  const bf16x8 *Wu, *Wo;  // weight images
  const bf16_t* A;        // [B][rows][d] attention output of the layer
  bf16_t* Y;              // [B][rows][d] next layer's input; nullable
  const float* sum_in;    // nullable = zero
  float* sum_out;         // nullable
  bf16_t* sum_rounded;    // nullable
  int B, rows, tiles_per_user, total_tiles;
};

template <int DH, int H>
__global__ __launch_bounds__(64 * H) void gated_block_kernel(GatedArgs a) {
  constexpr int D = DH * H, K1 = D / 16, MB = DH / 32;
  constexpr int PITCH = 2 * D + 16;  // bytes; the padding keeps the fragment reads free of bank conflicts
  constexpr int CPR = D / 8;         // 16-byte chunks per row
  constexpr int LW = DH / 16;        // 1 KiB loads per wave and tile: the H waves copy a tile of 32 rows together
  // Three tiles of 32 rows in LDS: the input rows X (fragments of the first product, then the residual), the
  // attention rows A (the gate's other factor; later the staged output rows), the gated rows Z.  Rows travel
  // between memory and LDS in whole 16-byte chunks, row-major and fully coalesced; the accumulator layout (a lane
  // owns a row, four adjacent columns per register quad) only ever touches LDS.
  __shared__ __attribute__((aligned(16))) unsigned char xs[32 * PITCH], as[32 * PITCH], zs[32 * PITCH];
  const int lane = threadIdx.x & 63, head = threadIdx.x >> 6;
  const int n = lane & 31, g = lane >> 5;
  bf16x8 wu[K1][MB], wo[K1][MB];
#pragma unroll
  for (int kk = 0; kk < K1; ++kk)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      wu[kk][mb] = a.Wu[((head * K1 + kk) * MB + mb) * 64 + lane];
      wo[kk][mb] = a.Wo[((head * K1 + kk) * MB + mb) * 64 + lane];
    }
  // this lane's chunks of a tile: (row, chunk) of piece j
  int crow[LW], cchunk[LW];
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int q = (head * LW + j) * 64 + lane;
    crow[j] = q / CPR, cchunk[j] = q % CPR;
  }
  bf16x8 rx[LW], ra[LW];
  auto request = [&](int tile) {  // rows at or past the user's length arrive as zeros
    const int b = tile / a.tiles_per_user, r0 = (tile - b * a.tiles_per_user) * 32;
    const int len = a.lens ? min(a.lens[b], a.rows) : a.rows;
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      bf16x8 vx, va;
#pragma unroll
      for (int t = 0; t < 8; ++t) vx[t] = va[t] = static_cast<__bf16>(0.f);
      const int row = r0 + crow[j];
      if (row < len) {
        vx = *reinterpret_cast<const bf16x8*>(a.X + b * a.x_user_stride + static_cast<int64_t>(row) * D + 8 * cchunk[j]);
        va = *reinterpret_cast<const bf16x8*>(a.A + (static_cast<int64_t>(b) * a.rows + row) * D + 8 * cchunk[j]);
      }
      rx[j] = vx, ra[j] = va;
    }
  };
  if (static_cast<int>(blockIdx.x) < a.total_tiles) request(blockIdx.x);
  for (int tile = blockIdx.x; tile < a.total_tiles; tile += gridDim.x) {
    const int b = tile / a.tiles_per_user, r0 = (tile - b * a.tiles_per_user) * 32;
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      *reinterpret_cast<bf16x8*>(xs + crow[j] * PITCH + cchunk[j] * 16) = rx[j];
      *reinterpret_cast<bf16x8*>(as + crow[j] * PITCH + cchunk[j] * 16) = ra[j];
    }
    __syncthreads();
    if (tile + static_cast<int>(gridDim.x) < a.total_tiles) request(tile + gridDim.x);  // in flight during this tile
    // P^T = Wu^T X^T: lane (row n, g), register 4j + r of block mb = column head DH + 32 mb + 8 j + 4 g + r
    f32x16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < K1; ++kk)
        acc[mb] = mfma32(wu[kk][mb], *reinterpret_cast<const bf16x8*>(xs + n * PITCH + (16 * kk + 8 * g) * 2), acc[mb]);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int at = n * PITCH + (head * DH + 32 * mb + 8 * j + 4 * g) * 2;
        const bf16x4 att = *reinterpret_cast<const bf16x4*>(as + at);
        bf16x4 z;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = acc[mb][4 * j + r];
          z[r] = static_cast<__bf16>(static_cast<float>(att[r]) * p * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-p * kLog2e)));
        }
        *reinterpret_cast<bf16x4*>(zs + at) = z;
      }
    __syncthreads();  // Z complete; nobody reads the attention rows any more
    f32x16 acc2[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc2[mb][i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < K1; ++kk)
        acc2[mb] = mfma32(wo[kk][mb], *reinterpret_cast<const bf16x8*>(zs + n * PITCH + (16 * kk + 8 * g) * 2), acc2[mb]);
    }
    const int row = r0 + n;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = head * DH + 32 * mb + 8 * j + 4 * g;
        if (a.Y != nullptr) {  // uniform: the output rows X + Y are staged where the attention rows were
          const bf16x4 xr = *reinterpret_cast<const bf16x4*>(xs + n * PITCH + col * 2);
          bf16x4 y;
#pragma unroll
          for (int r = 0; r < 4; ++r) y[r] = static_cast<__bf16>(static_cast<float>(xr[r]) + acc2[mb][4 * j + r]);
          *reinterpret_cast<bf16x4*>(as + n * PITCH + col * 2) = y;
        }
        if ((a.sum_out != nullptr || a.sum_rounded != nullptr) && row < a.rows) {
          const int64_t at = (static_cast<int64_t>(b) * a.rows + row) * D + col;
          f32x4 t = {0.f, 0.f, 0.f, 0.f};
          if (a.sum_in != nullptr) t = *reinterpret_cast<const f32x4*>(a.sum_in + at);
#pragma unroll
          for (int r = 0; r < 4; ++r) t[r] += acc2[mb][4 * j + r];
          if (a.sum_out != nullptr) *reinterpret_cast<f32x4*>(a.sum_out + at) = t;
          if (a.sum_rounded != nullptr) {
            bf16x4 tr;
#pragma unroll
            for (int r = 0; r < 4; ++r) tr[r] = static_cast<__bf16>(t[r]);
            *reinterpret_cast<bf16x4*>(a.sum_rounded + at) = tr;
          }
        }
      }
    __syncthreads();  // output rows staged; X and Z no longer needed
    if (a.Y != nullptr) {
      // (a row at or past the user's length arrived as zeros and has a zero attention row: its output is zero)
#pragma unroll
      for (int j = 0; j < LW; ++j)
        if (r0 + crow[j] < a.rows)
          *reinterpret_cast<bf16x8*>(a.Y + (static_cast<int64_t>(b) * a.rows + r0 + crow[j]) * D + 8 * cchunk[j]) =
              *reinterpret_cast<const bf16x8*>(as + crow[j] * PITCH + cchunk[j] * 16);
      __syncthreads();  // before the next tile's rows are parked over the staged ones
    }
  }
}

template <int DH, int H>
hipError_t launch_gated(const GatedArgs& p, hipStream_t s) {
  const int resident = (DH * H <= 128 ? 2 : 1) * compute_units();
  hipLaunchKernelGGL((gated_block_kernel<DH, H>), dim3(p.total_tiles < resident ? p.total_tiles : resident), dim3(64 * H), 0, s, p);
  return hipGetLastError();
}


// The history rows' part of an XOR layer in one pass (Eq. 7's O[S], then Eq. 8's gated block):
//   O[S] = SiLU(scale X W_Q K~^T) V~ / m per head,  Y = X + (O[S] * SiLU(X W_U)) W_O,
// each rounded where the kernels it takes the place of (queries_over_links_kernel, gated_block_kernel) store it, so with
// their bits.  One wave per head, all five stationary operands in registers; a tile of 32 rows goes through LDS for the
// first two products (which share its fragments), the gated rows and the output rows go through LDS once each.
// Two barriers a tile: the one that publishes a tile's rows also publishes the last tile's output rows, which the waves
// store during the next tile's products.
// What bounds it: memory traffic (one read and one write of the rows) and the vector ALUs (48 SiLUs per row and head at
// d/h = 32, m = 64) about equally.  B=8 N=16384 d=128 m=64, 67 MB: 17.5 + 21.3 us as two kernels, which also write and read
// O[S] and read the rows twice.
struct RowsArgs {
  const bf16_t* X;                 // [B][rows][d]
  const int32_t* lens;             // nullable; rows >= lens[b] count as zeros and are written as zeros
  const bf16x8 *Wq, *Wu, *Wo;      // weight images
  const bf16x8 *KA, *VA;           // key and value images of the links
  int64_t ka_user_frags, va_user_frags;
  bf16_t* Y;                       // [B][rows][d]
  int rows, tiles_per_user, total_tiles;
  float scale, inv_norm;           // scale >= 0 (a negative one is folded into the keys)
};

template <int DH, int M, int H>
__global__ __launch_bounds__(64 * H, DH * H == 128 && DH == 32 ? 2 : 1) void xor_rows_kernel(RowsArgs a) {
  constexpr int D = DH * H, K1 = D / 16, MB = DH / 32, K2 = DH / 16, LB = M / 32, K3 = M / 16;
  constexpr int PITCH = 2 * D + 16;  // bytes; the padding keeps the fragment reads free of bank conflicts
  constexpr int CPR = D / 8, LW = DH / 16;
  __shared__ __attribute__((aligned(16))) unsigned char xs[2][32 * PITCH], zs[32 * PITCH], ys[32 * PITCH];
  const int lane = threadIdx.x & 63, head = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int per_wg = (a.total_tiles + gridDim.x - 1) / gridDim.x;  // a contiguous run of tiles: few changes of user
  const int first = blockIdx.x * per_wg, last = min(first + per_wg, a.total_tiles);
  if (first >= last) return;  // uniform

  int lds_at[LW], row_of[LW];
  int64_t at[LW];
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int q = (head * LW + j) * 64 + lane;
    row_of[j] = q / CPR, lds_at[j] = q / CPR * PITCH + q % CPR * 16, at[j] = static_cast<int64_t>(q) * 8;
  }
  bf16x8 rx[LW];
  auto request = [&](int tile) {  // rows at or past the user's length arrive as zeros
    const int b = tile / a.tiles_per_user, r0 = (tile - b * a.tiles_per_user) * 32;
    const int len = a.lens ? min(a.lens[b], a.rows) : a.rows;
    const bf16_t* base = a.X + (static_cast<int64_t>(b) * a.rows + r0) * D;
    if (r0 + 32 <= len) {  // uniform
#pragma unroll
      for (int j = 0; j < LW; ++j) rx[j] = *reinterpret_cast<const bf16x8*>(base + at[j]);
    } else {
#pragma unroll
      for (int j = 0; j < LW; ++j) {
        bf16x8 v;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(0.f);
        if (r0 + row_of[j] < len) v = *reinterpret_cast<const bf16x8*>(base + at[j]);
        rx[j] = v;
      }
    }
  };
  request(first);
  bf16x8 wq[K1][MB], wu[K1][MB], wo[K1][MB], ka[K2][LB], va[K3][MB];
#pragma unroll
  for (int kk = 0; kk < K1; ++kk)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int f = ((head * K1 + kk) * MB + mb) * 64 + lane;
      // (W_U and W_O with their columns in the order of the value image, so that a lane gets 16 consecutive columns of a
      // block: out_col in place of the lane)
      const int fo = ((head * K1 + kk) * MB + mb) * 64 + out_col(n) + 32 * g;
      wq[kk][mb] = a.Wq[f], wu[kk][mb] = a.Wu[fo], wo[kk][mb] = a.Wo[fo];
    }
  auto load_user = [&](int b) {
    const bf16x8* k = a.KA + b * a.ka_user_frags + static_cast<int64_t>(head) * K2 * LB * 64 + lane;
    const bf16x8* v = a.VA + b * a.va_user_frags + static_cast<int64_t>(head) * K3 * MB * 64 + lane;
#pragma unroll
    for (int kk = 0; kk < K2; ++kk)
#pragma unroll
      for (int lb = 0; lb < LB; ++lb) ka[kk][lb] = k[(kk * LB + lb) * 64];
#pragma unroll
    for (int kk = 0; kk < K3; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) va[kk][mb] = v[(kk * MB + mb) * 64];
  };
  int cur_user = first / a.tiles_per_user;
  load_user(cur_user);

  auto store_rows = [&](int tile) {
    const int b = tile / a.tiles_per_user, r0 = (tile - b * a.tiles_per_user) * 32;
    bf16_t* base = a.Y + (static_cast<int64_t>(b) * a.rows + r0) * D;
    bf16x8 v[LW];
#pragma unroll
    for (int j = 0; j < LW; ++j) v[j] = *reinterpret_cast<const bf16x8*>(ys + lds_at[j]);
    if (r0 + 32 <= a.rows) {  // uniform
#pragma unroll
      for (int j = 0; j < LW; ++j) store_through(base, 32 * 2 * D, static_cast<int>(at[j]) * 2, v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < LW; ++j)
        if (r0 + row_of[j] < a.rows) *reinterpret_cast<bf16x8*>(base + at[j]) = v[j];
    }
  };
  const float c = a.scale * kLog2e, factor = a.inv_norm * a.scale;
  for (int tile = first; tile < last; ++tile) {
    const unsigned char* x_lds = xs[tile & 1];
#pragma unroll
    for (int j = 0; j < LW; ++j) *reinterpret_cast<bf16x8*>(xs[tile & 1] + lds_at[j]) = rx[j];
    lds_barrier();  // the tile's rows; the last tile's output rows
    if (tile + 1 < last) request(tile + 1);
    if (tile > first) store_rows(tile - 1);
    const int b = tile / a.tiles_per_user;
    if (b != cur_user) {  // uniform, rare: waited for right here, so that no other tile waits for its loads and stores
      load_user(b), cur_user = b;
#pragma unroll
      for (int kk = 0; kk < K2; ++kk)
#pragma unroll
        for (int lb = 0; lb < LB; ++lb) asm volatile("" : "+v"(ka[kk][lb]));
#pragma unroll
      for (int kk = 0; kk < K3; ++kk)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(va[kk][mb]));
    }
    // Q~^T = Wq_a^T X^T and P^T = Wu_a^T X^T
    f32x16 q[MB], p[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) q[mb][i] = p[mb][i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      const bf16x8 x = *reinterpret_cast<const bf16x8*>(x_lds + n * PITCH + (16 * kk + 8 * g) * 2);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) q[mb] = mfma32(wq[kk][mb], x, q[mb]), p[mb] = mfma32(wu[kk][mb], x, p[mb]);
    }
    bf16x8 qf[K2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) qf[2 * mb] = pack_half(q[mb], 0), qf[2 * mb + 1] = pack_half(q[mb], 1);
    // S^T = K~_a Q~^T, SiLU, O^T = V~_a^T SiLU(S)^T
    f32x16 s[LB], o[MB];
#pragma unroll
    for (int lb = 0; lb < LB; ++lb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[lb][i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < K2; ++kk)
#pragma unroll
      for (int lb = 0; lb < LB; ++lb) s[lb] = mfma32(ka[kk][lb], qf[kk], s[lb]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[mb][i] = 0.f;
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[lb][i] = s[lb][i] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-s[lb][i] * c));
      const bf16x8 p0 = pack_half(s[lb], 0), p1 = pack_half(s[lb], 1);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        o[mb] = mfma32(va[2 * lb][mb], p0, o[mb]);
        o[mb] = mfma32(va[2 * lb + 1][mb], p1, o[mb]);
      }
    }
    // register i of a block is column 16 g + i of it, in o, p and y
    const int own = n * PITCH + (head * DH + 16 * g) * 2;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        bf16x8 z;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float u = p[mb][8 * f + t], att = static_cast<float>(static_cast<__bf16>(o[mb][8 * f + t] * factor));
          z[t] = static_cast<__bf16>(att * u * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-u * kLog2e)));
        }
        *reinterpret_cast<bf16x8*>(zs + own + mb * 64 + f * 16) = z;
      }
    lds_barrier();  // Z complete; everybody has stored the last tile's output rows
    f32x16 y[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) y[mb][i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      const bf16x8 z = *reinterpret_cast<const bf16x8*>(zs + n * PITCH + (16 * kk + 8 * g) * 2);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) y[mb] = mfma32(wo[kk][mb], z, y[mb]);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const bf16x8 xr = *reinterpret_cast<const bf16x8*>(x_lds + own + mb * 64 + f * 16);
        bf16x8 v;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(static_cast<float>(xr[t]) + y[mb][8 * f + t]);
        *reinterpret_cast<bf16x8*>(ys + own + mb * 64 + f * 16) = v;
      }
  }
  lds_barrier();
  store_rows(last - 1);
}

template <int DH, int M, int H>
hipError_t launch_rows(const RowsArgs& p, hipStream_t s) {
  const int resident = (DH == 32 ? 2 : 1) * compute_units();
  hipLaunchKernelGGL((xor_rows_kernel<DH, M, H>), dim3(p.total_tiles < resident ? p.total_tiles : resident), dim3(64 * H), 0, s, p);
  return hipGetLastError();
}
template <int DH, int H>
hipError_t launch_rows(const RowsArgs& p, int m, hipStream_t s) {
  switch (m) {
    case 32: return launch_rows<DH, 32, H>(p, s);
    case 64: return launch_rows<DH, 64, H>(p, s);
    case 96: return launch_rows<DH, 96, H>(p, s);
  }
  return hipErrorInvalidValue;
}


// The link rows' part of an XOR layer: the gated block Y = (O[T] * SiLU(X W_U)) W_O, its place in the running sum and in the
// residual stream, and what the next layer's kernels need of the new rows X + Y: Q~ = . W_Q for the history kernel, K~ = . W_K
// and V~ = . W_V for the rows kernel, as the pack kernel would write them.  A workgroup takes 32 rows of one user, a wave per
// head-sized slice of columns.  Further workgroups write the next layer's images of W_U and W_O.
// What bounds it is latency: at B=8 m=64 d=128 it takes the place of a gated block of 4.8 and a pack launch of 4.0 us.
struct LinkArgs {
  const bf16_t* X;
  int64_t x_user_stride;
  const bf16x8 *Wu, *Wo, *Wq, *Wk, *Wv;  // weight images
  const bf16_t* A;                       // [B][m][d]
  bf16_t* Y;                             // [B][m][d]; null after the last layer, and with it all that follows
  const float* sum_in;
  float* sum_out;
  bf16_t* sum_rounded;
  bf16x8 *Q, *K, *V;                     // [B] images
  float sign;                            // of Q~ and K~
  const bf16_t* next_w[2];               // the next layer's W_U and W_O
  bf16x8* next_image[2];
  int m, tiles;                          // tiles: B m / 32
};

template <int DH, int H>
__global__ __launch_bounds__(64 * H) void xor_links_kernel(LinkArgs a) {
  constexpr int D = DH * H, K1 = D / 16, MB = DH / 32, PITCH = 2 * D + 16, CPR = D / 8, LW = DH / 16;
  if (static_cast<int>(blockIdx.x) >= a.tiles) {  // uniform: a wave per fragment of an image
    const int f = (blockIdx.x - a.tiles) * H + threadIdx.x / 64, job = f / (D * D / 512);
    if (job < 2) weight_fragment<DH>(a.next_w[job], a.next_image[job], D, f % (D * D / 512), threadIdx.x & 63);
    return;
  }
  __shared__ __attribute__((aligned(16))) unsigned char xs[32 * PITCH], as[32 * PITCH], zs[32 * PITCH];
  const int lane = threadIdx.x & 63, head = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int lbs = a.m / 32, b = blockIdx.x / lbs, lb = blockIdx.x % lbs;
  const int64_t row0 = static_cast<int64_t>(b) * a.m + 32 * lb;  // of all users' link rows
  const bool more = a.Y != nullptr;                              // uniform
  const bf16_t* X = a.X + b * a.x_user_stride + static_cast<int64_t>(32 * lb) * D;
  bf16x8 rx[LW], ra[LW], wu[K1][MB], wo[K1][MB], wq[K1][MB], wk[K1][MB], wv[K1][MB];
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int q = (head * LW + j) * 64 + lane;
    rx[j] = *reinterpret_cast<const bf16x8*>(X + q * 8);
    ra[j] = *reinterpret_cast<const bf16x8*>(a.A + row0 * D + q * 8);
  }
#pragma unroll
  for (int kk = 0; kk < K1; ++kk)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {  // (in the order that gives a lane 16 consecutive columns of a block)
      const int f = ((head * K1 + kk) * MB + mb) * 64 + out_col(n) + 32 * g;
      wu[kk][mb] = a.Wu[f], wo[kk][mb] = a.Wo[f];
    }
  if (more) {
#pragma unroll
    for (int kk = 0; kk < K1; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int f = ((head * K1 + kk) * MB + mb) * 64 + lane;
        wq[kk][mb] = a.Wq[f], wk[kk][mb] = a.Wk[f], wv[kk][mb] = a.Wv[f];
      }
  }
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int q = (head * LW + j) * 64 + lane, at = q / CPR * PITCH + q % CPR * 16;
    *reinterpret_cast<bf16x8*>(xs + at) = rx[j];
    *reinterpret_cast<bf16x8*>(as + at) = ra[j];
  }
  lds_barrier();
  auto rows_of = [&](const unsigned char* lds, int kk) { return *reinterpret_cast<const bf16x8*>(lds + n * PITCH + (16 * kk + 8 * g) * 2); };
  f32x16 p[MB], y[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) p[mb][i] = y[mb][i] = 0.f;
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) {
    const bf16x8 x = rows_of(xs, kk);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) p[mb] = mfma32(wu[kk][mb], x, p[mb]);
  }
  // register i of a block is column 16 g + i of it
  const int own = n * PITCH + (head * DH + 16 * g) * 2;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const bf16x8 att = *reinterpret_cast<const bf16x8*>(as + own + mb * 64 + f * 16);
      bf16x8 z;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float u = p[mb][8 * f + t];
        z[t] = static_cast<__bf16>(static_cast<float>(att[t]) * u * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-u * kLog2e)));
      }
      *reinterpret_cast<bf16x8*>(zs + own + mb * 64 + f * 16) = z;
    }
  lds_barrier();
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) {
    const bf16x8 z = rows_of(zs, kk);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) y[mb] = mfma32(wo[kk][mb], z, y[mb]);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int64_t at = (row0 + n) * D + head * DH + 32 * mb + 16 * g;
    if (more) {
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const bf16x8 xr = *reinterpret_cast<const bf16x8*>(xs + own + mb * 64 + f * 16);
        bf16x8 v;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = static_cast<__bf16>(static_cast<float>(xr[t]) + y[mb][8 * f + t]);
        *reinterpret_cast<bf16x8*>(as + own + mb * 64 + f * 16) = v;  // (where this lane alone has read)
        *reinterpret_cast<bf16x8*>(a.Y + at + 8 * f) = v;
      }
    }
    if (a.sum_in != nullptr) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(a.sum_in + at + 4 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[mb][4 * j + r] += t[r];
      }
    }
    if (a.sum_out != nullptr) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<f32x4*>(a.sum_out + at + 4 * j) = f32x4{y[mb][4 * j], y[mb][4 * j + 1], y[mb][4 * j + 2], y[mb][4 * j + 3]};
    }
    if (a.sum_rounded != nullptr) {
      *reinterpret_cast<bf16x8*>(a.sum_rounded + at) = pack_half(y[mb], 0);
      *reinterpret_cast<bf16x8*>(a.sum_rounded + at + 8) = pack_half(y[mb], 1);
    }
  }
  if (!more) return;
  lds_barrier();
  bf16x8 x[K1];
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) x[kk] = rows_of(as, kk);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    bf16x8 w[K1];
    auto of = [&](const bf16x8 (&all)[K1][MB]) {
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) w[kk] = all[kk][mb];
    };
    auto keys = [&](bf16x8* img) {
      f32x16 acc = project_block<K1>(w, x);
      if (a.sign < 0.f) acc = -acc;
      const int64_t frag = ((static_cast<int64_t>(b) * H + head) * (DH / 16) + 2 * mb) * lbs + lb;
      img[frag * 64 + lane] = pack_half(acc, 0);
      img[(frag + lbs) * 64 + lane] = pack_half(acc, 1);
    };
    of(wq), keys(a.Q);
    of(wk), keys(a.K);
    of(wv);
    const f32x16 acc = project_block<K1>(x, w);
    const int64_t frag = ((static_cast<int64_t>(b) * H + head) * (a.m / 16) + 2 * lb) * MB + mb;
    a.V[frag * 64 + out_rho(n) + 32 * g] = pack_half(acc, 0);
    a.V[(frag + MB) * 64 + out_rho(n) + 32 * g] = pack_half(acc, 1);
  }
}

template <int DH, int H>
hipError_t launch_links(const LinkArgs& p, hipStream_t s) {
  constexpr int kFragments = 2 * DH * H * DH * H / 512;
  const int images = p.next_w[0] != nullptr ? (kFragments + H - 1) / H : 0;
  hipLaunchKernelGGL((xor_links_kernel<DH, H>), dim3(p.tiles + images), dim3(64 * H), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t xor_links(const XorLinks& q, hipStream_t s) {
  auto image = [](void* p) { return static_cast<bf16x8*>(p); };
  LinkArgs p{static_cast<const bf16_t*>(q.X), q.x_user_stride, image(q.Wu_image), image(q.Wo_image), image(q.Wq_image), image(q.Wk_image),
             image(q.Wv_image), static_cast<const bf16_t*>(q.A), static_cast<bf16_t*>(q.Y), q.sum_in, q.sum_out,
             static_cast<bf16_t*>(q.sum_rounded), image(q.queries), image(q.keys), image(q.values), q.scale < 0.f ? -1.f : 1.f,
             {static_cast<const bf16_t*>(q.next_Wu), static_cast<const bf16_t*>(q.next_Wo)}, {image(q.next_Wu_image), image(q.next_Wo_image)},
             q.m, q.B * (q.m / 32)};
  const int dh = q.d / q.h;
  if (dh == 32) {
    switch (q.h) {
      case 1: return launch_links<32, 1>(p, s);
      case 2: return launch_links<32, 2>(p, s);
      case 4: return launch_links<32, 4>(p, s);
    }
  } else if (dh == 64) {
    switch (q.h) {
      case 1: return launch_links<64, 1>(p, s);
      case 2: return launch_links<64, 2>(p, s);
    }
  }
  return hipErrorInvalidValue;
}

// (five stationary operands: with d = 256, or with 128 links at d = 128, they do not fit the registers.  With 128 links at
// d <= 64 they would; those calls keep the kernels they have, and have not been measured on this one.)
bool xor_rows_supported(int d, int h, int m) { return queries_over_links_supported(d, h, m) && d <= 128 && m <= 96; }

hipError_t xor_rows(const XorRows& q, hipStream_t s) {
  const int tiles = (q.N + 31) / 32, dh = q.d / q.h;
  const int64_t frags = static_cast<int64_t>(q.m) * q.d / 8;
  RowsArgs p{static_cast<const bf16_t*>(q.X), q.lens, static_cast<const bf16x8*>(q.Wq_image), static_cast<const bf16x8*>(q.Wu_image),
             static_cast<const bf16x8*>(q.Wo_image), static_cast<const bf16x8*>(q.keys), static_cast<const bf16x8*>(q.values),
             q.per_user ? frags : 0, q.per_user ? frags : 0, static_cast<bf16_t*>(q.Y), q.N, tiles, tiles * q.B, fabsf(q.scale),
             1.f / static_cast<float>(q.m)};
  if (dh == 32) {
    switch (q.h) {
      case 1: return launch_rows<32, 1>(p, q.m, s);
      case 2: return launch_rows<32, 2>(p, q.m, s);
      case 4: return launch_rows<32, 4>(p, q.m, s);
    }
  } else if (dh == 64) {
    switch (q.h) {
      case 1: return launch_rows<64, 1>(p, q.m, s);
      case 2: return launch_rows<64, 2>(p, q.m, s);
    }
  }
  return hipErrorInvalidValue;
}

hipError_t gated_block(const GatedBlock& q, hipStream_t s) {
  if (q.B <= 0 || q.rows <= 0) return hipSuccess;
  const int tiles = (q.rows + 31) / 32;
  GatedArgs p{static_cast<const bf16_t*>(q.X), q.x_user_stride, q.lens, static_cast<const bf16x8*>(q.Wu_image),
              static_cast<const bf16x8*>(q.Wo_image), static_cast<const bf16_t*>(q.A), static_cast<bf16_t*>(q.Y), q.sum_in,
              q.sum_out, static_cast<bf16_t*>(q.sum_rounded), q.B, q.rows, tiles, tiles * q.B};
  const int dh = q.d / q.h;
  if (dh == 32) {
    switch (q.h) {
      case 1: return launch_gated<32, 1>(p, s);
      case 2: return launch_gated<32, 2>(p, s);
      case 4: return launch_gated<32, 4>(p, s);
      case 8: return launch_gated<32, 8>(p, s);
    }
  } else if (dh == 64) {
    switch (q.h) {
      case 1: return launch_gated<64, 1>(p, s);
      case 2: return launch_gated<64, 2>(p, s);
      case 4: return launch_gated<64, 4>(p, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace lime
