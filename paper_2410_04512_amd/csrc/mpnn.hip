// Learned warm start: a message-passing network over the collision graph,
// (F, v_prev) -> v_hat, used as the CG's initial guess (CG to the same
// tolerance still decides; the previous velocity is the fallback).
//
// Network (hidden width 64, three message-passing layers; the same
// definition as the FP64 oracle):
//   x_i = [F_i/sF, v_prev,i/sV],  e_p = [w/sW, n_ij] for CSR entry p = (i, j)
//   h = relu(x W_in + b_in)
//   per layer: z_p = h_i W_a + b_m + h_j W_b + e_p W_c; m_p = relu(z_p)
//              a_i = sum over row i of m_p;  h = h + relu([h, a] W_u + b_u)
//   out = h W_out + b_out,  v_hat = sV out
// The message MLP on [h_i, h_j, e_p] is split into the node products h W_a,
// h W_b (one node-level GEMM) and the per-edge gather-add, so the dense
// contractions run on MFMA and the per-edge part stays a bandwidth-bound
// gather instead of a 2m x 132 GEMM.
//
// Order: the network runs in the graph's internal (cell-list) vertex order,
// so a row's neighbours sit close in memory and the per-edge gathers mostly
// hit in L2; inputs are gathered and outputs scattered through the graph's
// permutation at the boundary.  The network is permutation-equivariant, so
// this changes only the order of roundings in its sums.
//
// Precision: FP32 master weights; every GEMM takes BF16 weights and BF16
// activations with FP32 accumulation (v_mfma_f32_16x16x16_bf16); the per-edge
// arithmetic uses the BF16-rounded W_c and b_m in FP32.  All reductions (row
// sums, column sums, split-K weight gradients) have a fixed order, so a step
// is bitwise reproducible.
#include "sgp_internal.h"

#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>

namespace {

constexpr int HID = 64, NL = 3;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

SGP_DEV unsigned short f2bf(float f)
{
    unsigned int b = __float_as_uint(f);
    b += 0x7FFFu + ((b >> 16) & 1u);   // round to nearest even
    return (unsigned short)(b >> 16);
}
SGP_DEV float bf2f(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

// flat parameter offsets (same order as the oracle's layout)
struct Layout {
    int64_t W_in, b_in, W_a[NL], W_b[NL], W_c[NL], b_m[NL], W_u[NL], b_u[NL], W_out, b_out, total;
};

Layout make_layout()
{
    Layout L;
    int64_t k = 0;
    L.W_in = k; k += 6 * HID;
    L.b_in = k; k += HID;
    for (int l = 0; l < NL; l++) {
        L.W_a[l] = k; k += HID * HID;
        L.W_b[l] = k; k += HID * HID;
        L.W_c[l] = k; k += 4 * HID;
        L.b_m[l] = k; k += HID;
        L.W_u[l] = k; k += 2 * HID * HID;
        L.b_u[l] = k; k += HID;
    }
    L.W_out = k; k += HID * 3;
    L.b_out = k; k += 3;
    L.total = k;
    return L;
}

// BF16 GEMM operands built from the master weights (K x N row-major, padded)
struct Packed {
    int64_t in16;           // W_in padded to 16 x 64
    int64_t ab[NL];         // [W_a | W_b]   64 x 128
    int64_t u[NL];          // W_u           128 x 64
    int64_t out16;          // W_out padded  64 x 16
    int64_t abT[NL];        // [W_a | W_b]^T 128 x 64
    int64_t uT[NL];         // W_u^T         64 x 128
    int64_t out16T;         // W_out^T pad   16 x 64
    int64_t total;
};

Packed make_packed()
{
    Packed p;
    int64_t k = 0;
    p.in16 = k; k += 16 * 64;
    for (int l = 0; l < NL; l++) { p.ab[l] = k; k += 64 * 128; }
    for (int l = 0; l < NL; l++) { p.u[l] = k; k += 128 * 64; }
    p.out16 = k; k += 64 * 16;
    for (int l = 0; l < NL; l++) { p.abT[l] = k; k += 128 * 64; }
    for (int l = 0; l < NL; l++) { p.uT[l] = k; k += 64 * 128; }
    p.out16T = k; k += 16 * 64;
    p.total = k;
    return p;
}

}   // namespace

struct sgp_mpnn_ {
    Layout L = make_layout();
    Packed PK = make_packed();
    DevBuf theta, m1, m2, grad, wbf, wrow;   // wrow: BF16-rounded master weights as FP32 (edge arithmetic)
    DevBuf wfrag;                            // weights of the fused layers (k_pack_frag)
    DevBuf act, efeat, part, vq;   // vq: v_hat and Gamma v_hat (FP64, canonical order)
    DevBuf irow, icol;                      // neighbour lists in the internal order (with efeat)
    const void *lists_of = nullptr;         // graph and version they were built for
    uint64_t lists_version = 0;
    double lists_sW = 0;
    double sF = 1, sV = 1, sW = 1;
    int64_t adam_t = 0;
    int64_t cap_n = 0, cap_e = 0;
};

namespace {

// ---------------------------------------------------------------- weight packing

__global__ void k_pack(const float *theta, Layout L, Packed P, unsigned short *wbf, float *wr)
{
    // one thread per packed element; wr receives every master weight rounded to BF16
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < L.total) wr[t] = bf2f(f2bf(theta[t]));
    if (t >= P.total) return;
    float v = 0.f;
    int64_t o = t;
    if (o < P.ab[0]) {   // in16: 16 x 64
        int r = (int)(o / 64), c = (int)(o % 64);
        v = r < 6 ? theta[L.W_in + r * 64 + c] : 0.f;
    } else if (o < P.u[0]) {
        int l = (int)((o - P.ab[0]) / (64 * 128));
        int64_t q = (o - P.ab[0]) % (64 * 128);
        int r = (int)(q / 128), c = (int)(q % 128);
        v = c < 64 ? theta[L.W_a[l] + r * 64 + c] : theta[L.W_b[l] + r * 64 + (c - 64)];
    } else if (o < P.out16) {
        int l = (int)((o - P.u[0]) / (128 * 64));
        int64_t q = (o - P.u[0]) % (128 * 64);
        v = theta[L.W_u[l] + q];
    } else if (o < P.abT[0]) {   // out16: 64 x 16
        int64_t q = o - P.out16;
        int r = (int)(q / 16), c = (int)(q % 16);
        v = c < 3 ? theta[L.W_out + r * 3 + c] : 0.f;
    } else if (o < P.uT[0]) {   // abT: 128 x 64
        int l = (int)((o - P.abT[0]) / (128 * 64));
        int64_t q = (o - P.abT[0]) % (128 * 64);
        int r = (int)(q / 64), c = (int)(q % 64);   // (r, c) of the transpose = (c, r) of [W_a | W_b]
        v = r < 64 ? theta[L.W_a[l] + c * 64 + r] : theta[L.W_b[l] + c * 64 + (r - 64)];
    } else if (o < P.out16T) {   // uT: 64 x 128
        int l = (int)((o - P.uT[0]) / (64 * 128));
        int64_t q = (o - P.uT[0]) % (64 * 128);
        int r = (int)(q / 128), c = (int)(q % 128);
        v = theta[L.W_u[l] + c * 64 + r];
    } else {   // out16T: 16 x 64
        int64_t q = o - P.out16T;
        int r = (int)(q / 64), c = (int)(q % 64);
        v = r < 3 ? theta[L.W_out + c * 3 + r] : 0.f;
    }
    wbf[o] = f2bf(v);
}

// The matrices of the fused layers in fragment order (k_layer reads a lane's
// four k-values of a 16 x 16 tile as one coalesced 8-byte load): per layer
// W_u (halves h and a, 4 x 4 tiles each) and the matrix of the product behind
// it, [W_a | W_b] of the next layer (4 x 8 tiles) or W_out (4 x 1).
constexpr int FRAG_U = 2 * 4 * 4 * 64, FRAG_N = 4 * 8 * 64, FRAG_LAYER = FRAG_U + FRAG_N;
__global__ void k_pack_frag(const unsigned short *wbf, Packed P, bf16x4 *out)
{
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= NL * FRAG_LAYER) return;
    const int l = t / FRAG_LAYER, e = t % FRAG_LAYER;
    const bool up = e < FRAG_U, last = l == NL - 1;
    const int f = up ? e : e - FRAG_U, lane = f & 63, NT = up ? 4 : last ? 1 : 8;
    const int kt = (f >> 6) / NT, nt = (f >> 6) % NT, N = 16 * NT;   // (W_u: 8 k-tiles, a's after h's)
    if (kt >= (up ? 8 : 4)) return;
    const unsigned short *B = wbf + (up ? P.u[l] : last ? P.out16 : P.ab[l + 1]);
    bf16x4 b;
    for (int k = 0; k < 4; k++) b[k] = (short)B[(16 * kt + 4 * (lane >> 4) + k) * N + 16 * nt + (lane & 15)];
    out[t] = b;
}

// ---------------------------------------------------------------- MFMA GEMM
//
// C[M x N] = A[M x K] B[K x N] (+ bias): A FP32 row-major (lda), B BF16
// row-major K x N, K = 16 KT and N multiples of 16 (<= 128).
// v_mfma_f32_16x16x16_bf16 lane layout (wave64): lane l holds
//   A[l % 16][4 (l / 16) + t], B[4 (l / 16) + t][l % 16], D[4 (l / 16) + t][l % 16], t = 0..3.
// B is staged in LDS in fragment order (a lane's four k-values adjacent, one
// 8-byte read); a wave converts the A fragments of its 16-row tile to BF16
// once and reuses them for every column tile.  A workgroup (4 waves) covers
// GEMM_ROWS rows (one 16-row tile per wave: more waves in flight than
// several tiles per wave, whose loads would wait for the previous tile).
constexpr int GEMM_ROWS = 64;

// What a product of the backward pass does with its result (BACK, N = 64, rows
// of 64 values): add1 + add2 (null: nothing) is added, the sum goes to C (null:
// not needed) and, where mask > 0, to dU, else 0 there.  Sums in the order of
// passes of their own, which read and wrote the rows once more each (60k cells:
// 13 us a mask, 10 us an addition).
struct GemmBack {
    const float *add1, *add2;
    int64_t ld2;
    const float *mask;
    float *dU;
};

template <int KT, bool BACK>
__global__ __launch_bounds__(256) void k_gemm(const float *A, int64_t lda, const unsigned short *B, float *C,
                                              int64_t ldc, int64_t M, int N, const float *bias, float *R, GemmBack bk)
{
    __shared__ bf16x4 sB[KT * 8 * 64];
    const int NT = N >> 4;
    for (int e = threadIdx.x; e < KT * NT * 64; e += 256) {
        const int ln = e & 63, tile = e >> 6, kt = tile / NT, nt = tile % NT;
        bf16x4 b;
        for (int t = 0; t < 4; t++) b[t] = (short)B[(16 * kt + 4 * (ln >> 4) + t) * N + 16 * nt + (ln & 15)];
        sB[e] = b;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    for (int it = 0; it < GEMM_ROWS / 64; it++) {
        const int64_t r0 = (int64_t)blockIdx.x * GEMM_ROWS + 64 * it + 16 * wv;
        if (r0 >= M) break;
        // every load of the tile before any store, unconditional (rows past
        // M read row M-1 and are not stored): a load behind a store, or in a
        // branch, would wait for it
        const int64_t arow = min(r0 + lr, M - 1);
        float4 av[KT];
#pragma unroll
        for (int kt = 0; kt < KT; kt++) av[kt] = *(const float4 *)(A + arow * lda + 16 * kt + 4 * lg);
        float bv[8], c1[BACK ? 4 : 1][4], c2[BACK ? 4 : 1][4], mk[BACK ? 4 : 1][4];
#pragma unroll
        for (int nt = 0; nt < 8; nt++) bv[nt] = bias && nt < NT ? bias[16 * nt + lr] : 0.f;
        if (BACK) {
#pragma unroll
            for (int nt = 0; nt < 4; nt++)
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const int64_t row = min(r0 + 4 * lg + t, M - 1);
                    const int c = 16 * nt + lr;
                    mk[nt][t] = bk.mask[row * 64 + c];
                    c1[nt][t] = bk.add1 ? bk.add1[row * 64 + c] : 0.f;
                    c2[nt][t] = bk.add1 ? bk.add2[row * bk.ld2 + c] : 0.f;
                }
        }
        keep_loads_above();
        bf16x4 a[KT];
#pragma unroll
        for (int kt = 0; kt < KT; kt++) {
            a[kt][0] = (short)f2bf(av[kt].x);
            a[kt][1] = (short)f2bf(av[kt].y);
            a[kt][2] = (short)f2bf(av[kt].z);
            a[kt][3] = (short)f2bf(av[kt].w);
        }
#pragma unroll
        for (int nt = 0; nt < (BACK ? 4 : 8); nt++) {
            if (!BACK && nt >= NT) break;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < KT; kt++)
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[kt], sB[(kt * NT + nt) * 64 + lane], acc, 0, 0, 0);
            for (int t = 0; t < 4; t++) {
                const int64_t row = r0 + 4 * lg + t;
                if (row >= M) continue;
                const float v = acc[t] + bv[nt];
                if (BACK) {
                    const float o = bk.add1 ? (c1[nt][t] + c2[nt][t]) + v : v;
                    if (C) C[row * 64 + 16 * nt + lr] = o;
                    bk.dU[row * 64 + 16 * nt + lr] = mk[nt][t] > 0.f ? o : 0.f;
                    continue;
                }
                C[row * ldc + 16 * nt + lr] = v;
                if (R) R[row * ldc + 16 * nt + lr] = fmaxf(v, 0.f);
            }
        }
    }
}

// Weight-gradient partials: workgroup g's [A | A2]^T D (K x N, the row index
// the reduction dimension of the MFMAs) over its share of the 16-row blocks,
// then its column sums of D (N values, FP32).  A lane's four reduction-index
// values are four rows of one column, so the fragments come straight from
// global memory (64-byte segments; the other tiles of the block read the rest of
// the same lines): no LDS, no barrier, and each wave walks blocks of its own,
// all loads of a block ahead of its MFMAs.  A wave keeps all K x N sums; the
// workgroup adds its four waves in LDS.  Bound by memory: 60k rows, 64 x 128:
// 118 -> 21 us (before, 512-row chunks through LDS: 118 workgroups, each
// waiting for one slab at a time).  Every sum has a fixed order.
constexpr int AT_GRID = 256;

template <int KT1, int KT2, int NT>
__global__ __launch_bounds__(256) void k_gemm_at(const float *A, int64_t lda, const float *A2, int64_t lda2,
                                                 const float *D, int64_t ldd, int64_t M, float *part)
{
    constexpr int KT = KT1 + KT2, K = 16 * KT, N = 16 * NT;
    __shared__ float sh[K * N + N];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
    f32x4 acc[KT][NT];
    float cs[NT];
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
        cs[nt] = 0.f;
#pragma unroll
        for (int kt = 0; kt < KT; kt++) acc[kt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const int64_t nblk = (M + 15) / 16, step = 4 * (int64_t)gridDim.x;
    for (int64_t blk = 4 * (int64_t)blockIdx.x + wv; blk < nblk; blk += step) {
        float av[KT][4], dv[NT][4];
        const int64_t r0 = 16 * blk + 4 * lg;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int64_t r = min(r0 + t, M - 1);
#pragma unroll
            for (int nt = 0; nt < NT; nt++) dv[nt][t] = D[r * ldd + 16 * nt + lr];
#pragma unroll
            for (int kt = 0; kt < KT1; kt++) av[kt][t] = A[r * lda + 16 * kt + lr];
#pragma unroll
            for (int kt = 0; kt < KT2; kt++) av[KT1 + kt][t] = A2[r * lda2 + 16 * kt + lr];
        }
        keep_loads_above();
        bf16x4 a[KT];
#pragma unroll
        for (int kt = 0; kt < KT; kt++)
#pragma unroll
            for (int t = 0; t < 4; t++) a[kt][t] = (short)f2bf(r0 + t < M ? av[kt][t] : 0.f);
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            bf16x4 d;
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const float v = r0 + t < M ? dv[nt][t] : 0.f;
                cs[nt] += v;
                d[t] = (short)f2bf(v);
            }
#pragma unroll
            for (int kt = 0; kt < KT; kt++)
                acc[kt][nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[kt], d, acc[kt][nt], 0, 0, 0);
        }
    }
    // the four waves in order, then out
    for (int w = 0; w < 4; w++) {
        if (wv == w) {
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                float c = cs[nt];
                c += __shfl_xor(c, 16, 64);
                c += __shfl_xor(c, 32, 64);
                if (lg == 0) sh[K * N + 16 * nt + lr] = w ? sh[K * N + 16 * nt + lr] + c : c;
#pragma unroll
                for (int kt = 0; kt < KT; kt++)
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        float *o = sh + (16 * kt + 4 * lg + t) * N + 16 * nt + lr;
                        *o = w ? *o + acc[kt][nt][t] : acc[kt][nt][t];
                    }
            }
        }
        __syncthreads();
    }
    float *P = part + (int64_t)blockIdx.x * (K * N + N);
    for (int t = threadIdx.x; t < K * N + N; t += 256) P[t] = sh[t];
}

// Where a sum of partials goes in the gradient: value (r, c) of the K x N
// product to w0[r ld + c] for c < c1 and to w1[r ld + c - c1] for c1 <= c < c2
// (rows below `rows` only), the column sums of columns below c1 to b (if any).
struct GradOut {
    float *w0, *w1, *b;
    int K, N, rows, c1, c2, ld;
};

// Fixed-order sum of G partial vectors of length L: 64 values per workgroup,
// its 16 waves a contiguous run of partials each (eight loads in flight), the
// runs added in order, and each sum stored where it belongs: one launch instead
// of two sums and up to three copies.
constexpr int RED_WAVES = 16;
__global__ __launch_bounds__(64 * RED_WAVES) void k_red_out(const float *part, int G, int L, GradOut o)
{
    __shared__ float sh[RED_WAVES][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane, cc = min(c, L - 1);
    const int per = (G + RED_WAVES - 1) / RED_WAVES, p0 = min(wv * per, G), p1 = min(p0 + per, G);
    float acc = 0.f;
    for (int p = p0; p < p1; p += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = part[(int64_t)min(p + u, p1 - 1) * L + cc];
#pragma unroll
        for (int u = 0; u < 8; u++) acc += p + u < p1 ? v[u] : 0.f;
    }
    sh[wv][lane] = acc;
    __syncthreads();
    if (wv != 0 || c >= L) return;
    float s = 0.f;
    for (int w = 0; w < RED_WAVES; w++) s += sh[w][lane];
    const int r = c / o.N, k = c % o.N;
    if (r >= o.K) {
        if (o.b && k < o.c1) o.b[k] = s;
    } else if (r < o.rows) {
        if (k < o.c1) o.w0[r * o.ld + k] = s;
        else if (k < o.c2) o.w1[r * o.ld + k - o.c1] = s;
    }
}

// ---------------------------------------------------------------- elementwise

// node features of internal vertex i = graph vertex perm[i]
__global__ void k_input(int64_t n, const int32_t *perm, const double *F, const double *vp, float sF, float sV,
                        float *x16)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    float *x = x16 + 16 * i;
    for (int a = 0; a < 3; a++) {
        x[a] = (float)(F[3 * u + a] / sF);
        x[3 + a] = (float)(vp[3 * u + a] / sV);
    }
    for (int a = 6; a < 16; a++) x[a] = 0.f;
}

// neighbour count of internal row i
__global__ void k_int_deg(int64_t n, const int32_t *perm, const int32_t *rowptr, int32_t *deg)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t u = perm[i];
    deg[i] = rowptr[u + 1] - rowptr[u];
}

// internal neighbour lists (the graph's row order kept within a row) and the
// edge features e_p = [w/sW, n], n = (r_i - r_j)/d = -u_e when i < j in the
// graph's numbering, +u_e otherwise.  16 threads per row, one entry each.
__global__ void k_int_entries(int64_t n, const int32_t *perm, const int32_t *inv, const int32_t *rowptr,
                              const int32_t *col, const int32_t *ent_edge, const double4 *wu, float sW,
                              const int32_t *irow, int32_t *icol, float4 *ef)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t >> 4;
    if (i >= n) return;
    const int32_t u = perm[i];
    const int32_t b = rowptr[u], e = rowptr[u + 1], k0 = irow[i];
    for (int32_t c = (int32_t)(t & 15); c < e - b; c += 16) {
        const int32_t j = col[b + c];
        const double4 q = wu[ent_edge[b + c]];
        const float sg = (u < j) ? -1.f : 1.f;
        icol[k0 + c] = inv[j];
        ef[k0 + c] = make_float4((float)(q.x / sW), sg * (float)q.y, sg * (float)q.z, sg * (float)q.w);
    }
}

// ---------------------------------------------------------------- messages (16 lanes per row, four features per lane)

// A row's 16 lanes load the columns and edge features of 16 of its entries at
// once, a lane each, and hand them round by DPP row broadcasts; the neighbour
// gathers, which wait for the columns, go six, six and four at a time, then the
// arithmetic in entry order, as in a plain loop.  Every lane loading every
// entry's column and features (eight entries at a time, two waits per eight)
// took twice the load instructions and 64 more registers: forward, 200k cells,
// 93 -> 64 us.
template <int U>
SGP_DEV int row_bcast(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + U, 0xf, 0xf, false);
}
template <int U>
SGP_DEV float4 row_bcast(const float4 &v)
{
    return make_float4(__int_as_float(row_bcast<U>(__float_as_int(v.x))), __int_as_float(row_bcast<U>(__float_as_int(v.y))),
                       __int_as_float(row_bcast<U>(__float_as_int(v.z))), __int_as_float(row_bcast<U>(__float_as_int(v.w))));
}

template <class F, int... U>
SGP_DEV void static_for(std::integer_sequence<int, U...>, F f)
{
    (f(std::integral_constant<int, U>()), ...);
}

// entries OFF .. OFF + N - 1 of the lanes' 16 (cnt of them the row's, the rest
// copies of its last): get(column) for all, then use(features, value) in order
template <int OFF, int N, class Get, class Use>
SGP_DEV void msg_group(int32_t jl, const float4 &el, int cnt, Get get, Use use)
{
    using Idx = std::make_integer_sequence<int, N>;
    decltype(get(0)) v[N];
    static_for(Idx(), [&](auto u) { v[u] = get(row_bcast<OFF + decltype(u)::value>(jl)); });
    keep_loads_above();
    static_for(Idx(), [&](auto u) {
        const float4 e = row_bcast<OFF + decltype(u)::value>(el);
        if (OFF + decltype(u)::value < cnt) use(e, v[u]);
    });
}

// a row's up to 16 entries from p on, whose columns and features the lanes hold
template <class Get, class Use>
SGP_DEV void msg_16(int32_t p, int32_t re, int32_t jl, const float4 &el, Get get, Use use)
{
    const int cnt = re - p < 16 ? re - p : 16;
    if (cnt > 0) msg_group<0, 6>(jl, el, cnt, get, use);
    if (cnt > 6) msg_group<6, 6>(jl, el, cnt, get, use);
    if (cnt > 12) msg_group<12, 4>(jl, el, cnt, get, use);
}

template <class Get, class Use>
SGP_DEV void msg_row(int32_t p, int32_t re, const int32_t *col, const float4 *ef, Get get, Use use)
{
    for (; p < re; p += 16) {
        const int32_t pc = min(p + (int)(threadIdx.x & 15), re - 1);
        const int32_t jl = col[pc];
        const float4 el = ef[pc];
        msg_16(p, re, jl, el, get, use);
    }
}

// One layer of the network in one pass: the messages a of 16 rows per wave, U =
// [h, a] W_u + b_u as two K = 64 products (h's plus the bias, then a's, added in
// that order), h' = h + relu(U), and the product behind it, h' [W_a | W_b] of
// the next layer or h' W_out.  a and h' pass from one step to the next in LDS
// (fragments want a lane's k-values of one row, results come as rows of a
// column).  a, U (null: no backward pass follows) and h' (null: after the last
// layer) are stored for others.  Bound by the gathers of the messages (64 us
// alone at 200k rows); as four passes over memory (messages, update, product)
// a layer of 200k rows took 129 us instead of 116, the last one 113 instead of
// 79.  Four waves per SIMD fit 128 registers; with three it took 133.
// Rows past n are computed from row n - 1 and not stored.
constexpr int LAYER_ROWS = 64, LAYER_LD = 68;   // (16-byte rows, four banks apart)
template <int NT2>
__global__ __launch_bounds__(256, 4) void k_layer(int64_t n, const int32_t *rowptr, const int32_t *col, const float4 *ef,
                                               const float *PQ, const float *bm, const float *Wc, const float *H,
                                               const bf16x4 *Bu, const float *bias, const bf16x4 *B2, float *agg,
                                               float *U, float *Hn, float *C, int64_t ldc)
{
    constexpr int KT = 4, NT = 4, N = 64;
    __shared__ float st[4][16][LAYER_LD], sth[4][16][LAYER_LD];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int lr = lane & 15, lg = lane >> 4, f = 4 * lr;
    const int64_t r0 = xcd_block(blockIdx.x, gridDim.x) * LAYER_ROWS + 16 * wv;
    if (r0 >= n) return;
    float(*s)[LAYER_LD] = st[wv], (*sh)[LAYER_LD] = sth[wv];
    // messages: 16 lanes per row, four features per lane, rows 4 k + lg in turn;
    // the ranges, then the first 16 entries' columns and features of all four
    int32_t p0[4], p1[4], jl[4];
    float4 el[4], pq[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int64_t i = min(r0 + 4 * k + lg, n - 1);
        p0[k] = rowptr[i];
        p1[k] = rowptr[i + 1];
        pq[k] = *(const float4 *)(PQ + i * 128 + f);
    }
    const float4 b4 = *(const float4 *)(bm + f);
    const float4 w0 = *(const float4 *)(Wc + f), w1 = *(const float4 *)(Wc + 64 + f);
    const float4 w2 = *(const float4 *)(Wc + 128 + f), w3 = *(const float4 *)(Wc + 192 + f);
    keep_loads_above();
#pragma unroll
    for (int k = 0; k < 4; k++) {
        // (a row without entries: entry 0, or the rows' end less one, unused)
        const int32_t pc = max(min(p0[k] + lr, p1[k] - 1), 0);
        jl[k] = p1[k] > p0[k] ? col[pc] : 0;
        el[k] = p1[k] > p0[k] ? ef[pc] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const float P0 = pq[k].x + b4.x, P1 = pq[k].y + b4.y, P2 = pq[k].z + b4.z, P3 = pq[k].w + b4.w;
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
        auto get = [&](int32_t j) { return *(const float4 *)(PQ + (int64_t)j * 128 + 64 + f); };
        auto use = [&](const float4 &e, const float4 &q) {
            a0 += fmaxf(P0 + q.x + (e.x * w0.x + e.y * w1.x + e.z * w2.x + e.w * w3.x), 0.f);
            a1 += fmaxf(P1 + q.y + (e.x * w0.y + e.y * w1.y + e.z * w2.y + e.w * w3.y), 0.f);
            a2 += fmaxf(P2 + q.z + (e.x * w0.z + e.y * w1.z + e.z * w2.z + e.w * w3.z), 0.f);
            a3 += fmaxf(P3 + q.w + (e.x * w0.w + e.y * w1.w + e.z * w2.w + e.w * w3.w), 0.f);
        };
        msg_16(p0[k], p1[k], jl[k], el[k], get, use);
        if (p1[k] - p0[k] > 16) msg_row(p0[k] + 16, p1[k], col, ef, get, use);
        const float4 a = make_float4(a0, a1, a2, a3);
        *(float4 *)&s[4 * k + lg][f] = a;
        const int64_t i = r0 + 4 * k + lg;
        if (agg && i < n) *(float4 *)(agg + i * 64 + f) = a;
    }
    // update: the fragments of h and a, and h at the lane's output positions,
    // all from LDS (whole rows in and out of memory: a lane's four values of
    // one column are four rows, 64 bytes a row and instruction)
    float4 hr[4];
#pragma unroll
    for (int k = 0; k < 4; k++) hr[k] = *(const float4 *)(H + min(r0 + 4 * k + lg, n - 1) * 64 + f);
    float bv[NT];
#pragma unroll
    for (int nt = 0; nt < NT; nt++) bv[nt] = bias[16 * nt + lr];
#pragma unroll
    for (int k = 0; k < 4; k++) *(float4 *)&sh[4 * k + lg][f] = hr[k];
    lds_wave_barrier();
    auto frag = [](const float4 &v) {
        bf16x4 b;
        b[0] = (short)f2bf(v.x);
        b[1] = (short)f2bf(v.y);
        b[2] = (short)f2bf(v.z);
        b[3] = (short)f2bf(v.w);
        return b;
    };
    bf16x4 ah[KT], aa[KT];
#pragma unroll
    for (int kt = 0; kt < KT; kt++) {
        ah[kt] = frag(*(const float4 *)&sh[lr][16 * kt + 4 * lg]);
        aa[kt] = frag(*(const float4 *)&s[lr][16 * kt + 4 * lg]);
    }
    lds_wave_barrier();
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
        f32x4 acc1 = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < KT; kt++) {
            acc1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah[kt], Bu[(kt * NT + nt) * 64 + lane], acc1, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aa[kt], Bu[((KT + kt) * NT + nt) * 64 + lane], acc2, 0, 0,
                                                             0);
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int64_t row = r0 + 4 * lg + t, o = row * N + 16 * nt + lr;
            const float u = (acc1[t] + bv[nt]) + (acc2[t] + 0.f);
            if (U && row < n) U[o] = u;
            s[4 * lg + t][16 * nt + lr] = sh[4 * lg + t][16 * nt + lr] + fmaxf(u, 0.f);
        }
    }
    lds_wave_barrier();
    // whole rows of LDS to memory
    auto store_rows = [&](const float(*src)[LAYER_LD], float *dst, int64_t ld) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int64_t i = r0 + 4 * k + lg;
            if (i < n) *(float4 *)(dst + i * ld + f) = *(const float4 *)&src[4 * k + lg][f];
        }
    };
    if (Hn) store_rows(s, Hn, 64);
    // the product behind it
    bf16x4 an[KT];
#pragma unroll
    for (int kt = 0; kt < KT; kt++) an[kt] = frag(*(const float4 *)&s[lr][16 * kt + 4 * lg]);
#pragma unroll
    for (int nt = 0; nt < NT2; nt++) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < KT; kt++)
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(an[kt], B2[(kt * NT2 + nt) * 64 + lane], acc, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int64_t row = r0 + 4 * lg + t;
            if (NT2 >= 4)
                sh[4 * lg + t][16 * (nt & 3) + lr] = acc[t] + 0.f;
            else if (row < n)
                C[row * ldc + 16 * nt + lr] = acc[t] + 0.f;
        }
        if (NT2 >= 4 && (nt & 3) == 3) {   // four tiles make 64 columns of the rows
            lds_wave_barrier();
            store_rows(sh, C + 16 * (nt - 3), ldc);
            lds_wave_barrier();
        }
    }
}

// dP_i = sum over row i of dz_p, dz_p = da_i [z_p > 0]; per-workgroup partials
// of e_p^T dz_p (4 x 64).  Rows are walked as in the forward messages (60k
// rows: 34 us, and 26 in k_msg_bwd_q; with every lane loading every entry's
// column and features 38 and 28, one wave per row with loads behind branches 74
// and 63).  The grid is fixed (at most MSG_BWD_GRID workgroups);
// workgroup b (in XCD-contiguous order) walks its own contiguous run of 16-row
// blocks in order.
constexpr int MSG_BWD_GRID = 2048;

__global__ __launch_bounds__(256) void k_msg_bwd_p(int64_t n, const int32_t *rowptr, const int32_t *col,
                                                   const float4 *ef, const float *PQ, const float *bm,
                                                   const float *Wc, const float *da, int64_t ldda, float *dPQ,
                                                   float *wc_part)
{
    __shared__ float sw[4][256];
    const int wv = threadIdx.x >> 6, f = 4 * (threadIdx.x & 15);
    const float4 w0 = *(const float4 *)(Wc + f), w1 = *(const float4 *)(Wc + 64 + f);
    const float4 w2 = *(const float4 *)(Wc + 128 + f), w3 = *(const float4 *)(Wc + 192 + f);
    const float4 b4 = *(const float4 *)(bm + f);
    float g[4][4];
    for (int a = 0; a < 4; a++)
        for (int k = 0; k < 4; k++) g[a][k] = 0.f;
    const int64_t nblk = (n + 15) / 16, per = (nblk + gridDim.x - 1) / gridDim.x;
    const int64_t k0 = xcd_block(blockIdx.x, gridDim.x) * per;
    const int64_t k1 = k0 + per < nblk ? k0 + per : nblk;
    for (int64_t blk = k0; blk < k1; blk++) {
        const int64_t i = blk * 16 + (threadIdx.x >> 4);
        if (i >= n) continue;
        const float4 pq = *(const float4 *)(PQ + i * 128 + f), d4 = *(const float4 *)(da + i * ldda + f);
        const float P[4] = {pq.x + b4.x, pq.y + b4.y, pq.z + b4.z, pq.w + b4.w}, dai[4] = {d4.x, d4.y, d4.z, d4.w};
        float dp[4] = {0.f, 0.f, 0.f, 0.f};
        msg_row(
            rowptr[i], rowptr[i + 1], col, ef,
            [&](int32_t j) { return *(const float4 *)(PQ + (int64_t)j * 128 + 64 + f); },
            [&](const float4 &e, const float4 &q) {
                const float z[4] = {P[0] + q.x + (e.x * w0.x + e.y * w1.x + e.z * w2.x + e.w * w3.x),
                                    P[1] + q.y + (e.x * w0.y + e.y * w1.y + e.z * w2.y + e.w * w3.y),
                                    P[2] + q.z + (e.x * w0.z + e.y * w1.z + e.z * w2.z + e.w * w3.z),
                                    P[3] + q.w + (e.x * w0.w + e.y * w1.w + e.z * w2.w + e.w * w3.w)};
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const float dz = z[k] > 0.f ? dai[k] : 0.f;
                    dp[k] += dz;
                    g[0][k] += e.x * dz;
                    g[1][k] += e.y * dz;
                    g[2][k] += e.z * dz;
                    g[3][k] += e.w * dz;
                }
            });
        *(float4 *)(dPQ + i * 128 + f) = make_float4(dp[0], dp[1], dp[2], dp[3]);
    }
    // a wave's four row groups, then the four waves
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int k = 0; k < 4; k++) {
            float v = g[a][k];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if ((threadIdx.x & 63) < 16) sw[wv][64 * a + f + k] = v;
        }
    __syncthreads();
    const int t = threadIdx.x;   // 256 = 4 x 64 outputs
    wc_part[(int64_t)blockIdx.x * 256 + t] = (sw[0][t] + sw[1][t]) + (sw[2][t] + sw[3][t]);
}

// dQ_j = sum over the entries (i, j) of column j of dz: walked as row j's
// entries (j, i) with the twin's features e = [w, -n]
__global__ __launch_bounds__(256) void k_msg_bwd_q(int64_t n, const int32_t *rowptr, const int32_t *col,
                                                   const float4 *ef, const float *PQ, const float *bm,
                                                   const float *Wc, const float *da, int64_t ldda, float *dPQ)
{
    struct Two {
        float4 p, d;
    };
    const int64_t j = xcd_block(blockIdx.x, gridDim.x) * 16 + (threadIdx.x >> 4);
    const int f = 4 * (threadIdx.x & 15);
    if (j >= n) return;
    const float4 q4 = *(const float4 *)(PQ + j * 128 + 64 + f), b4 = *(const float4 *)(bm + f);
    const float4 w0 = *(const float4 *)(Wc + f), w1 = *(const float4 *)(Wc + 64 + f);
    const float4 w2 = *(const float4 *)(Wc + 128 + f), w3 = *(const float4 *)(Wc + 192 + f);
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    msg_row(
        rowptr[j], rowptr[j + 1], col, ef,
        [&](int32_t i) {
            return Two{*(const float4 *)(PQ + (int64_t)i * 128 + f), *(const float4 *)(da + (int64_t)i * ldda + f)};
        },
        [&](const float4 &e, const Two &v) {
            const float4 P = v.p, d = v.d;
            a0 += (P.x + b4.x) + q4.x + (e.x * w0.x - e.y * w1.x - e.z * w2.x - e.w * w3.x) > 0.f ? d.x : 0.f;
            a1 += (P.y + b4.y) + q4.y + (e.x * w0.y - e.y * w1.y - e.z * w2.y - e.w * w3.y) > 0.f ? d.y : 0.f;
            a2 += (P.z + b4.z) + q4.z + (e.x * w0.z - e.y * w1.z - e.z * w2.z - e.w * w3.z) > 0.f ? d.z : 0.f;
            a3 += (P.w + b4.w) + q4.w + (e.x * w0.w - e.y * w1.w - e.z * w2.w - e.w * w3.w) > 0.f ? d.w : 0.f;
        });
    *(float4 *)(dPQ + j * 128 + 64 + f) = make_float4(a0, a1, a2, a3);
}

// loss = mean (out - v/sV)^2 over 3n values; dout16 = 2 (out - v/sV)/(3n) in columns 0..2
__global__ __launch_bounds__(256) void k_loss(int64_t n, const int32_t *perm, const float *out16, const float *bout,
                                              const double *v, float sV, float *dout16, double *part)
{
    __shared__ double sh[256];
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    if (i < n) {
        for (int a = 0; a < 16; a++) {
            float d = 0.f;
            if (a < 3) {
                d = (out16[16 * i + a] + bout[a]) - (float)(v[3 * (int64_t)perm[i] + a] / sV);
                s += (double)d * (double)d;
                d = 2.f * d / (float)(3 * n);
            }
            dout16[16 * i + a] = d;
        }
    }
    s = block_sum_256(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// energy loss sums per block: (v_hat . Gamma v_hat, v_hat . F, v . F); v == nullptr
// leaves the third at zero (the warm-start energies need only the first two)
__global__ __launch_bounds__(256) void k_energy_parts(int64_t len, const double *vh, const double *q, const double *F,
                                                      const double *v, double *part)
{
    __shared__ double sh[256];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < len; t += (int64_t)gridDim.x * 256) {
        a += vh[t] * q[t];
        b += vh[t] * F[t];
        if (v) c += v[t] * F[t];
    }
    a = block_sum_256(a, sh);
    b = block_sum_256(b, sh);
    c = block_sum_256(c, sh);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x] = a;
        part[3 * blockIdx.x + 1] = b;
        part[3 * blockIdx.x + 2] = c;
    }
}

// s[k] = sum over blocks of part[3 b + k], in block order
__global__ void k_sum3(const double *part, int np, double *s)
{
    __shared__ double sh[256];
    for (int k = 0; k < 3; k++) {
        double a = 0.0;
        for (int b = threadIdx.x; b < np; b += 256) a += part[3 * b + k];
        a = block_sum_256(a, sh);
        if (threadIdx.x == 0) s[k] = a;
    }
}

// d loss / d out = 2 sV (Gamma v_hat - F) / (v . F) in columns 0..2
__global__ void k_energy_dout(int64_t n, const int32_t *perm, const double *q, const double *F, double sV,
                              const double *s, float *dout16)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const double scale = 2.0 * sV / s[2];
    for (int a = 0; a < 16; a++)
        dout16[16 * i + a] = a < 3 ? (float)(scale * (q[3 * u + a] - F[3 * u + a])) : 0.f;
}

// The start of lowest energy E(x) = 0.5 x' Gamma x - x' F among v_prev, the
// network's guess and zero (E = 0), in that order of preference on ties
// (0: v_prev, 1: the network, 2: zero).  Lower energy is the smaller
// Gamma-norm error, since E(x) - E(v) = 0.5 ||x - v||^2_Gamma.
SGP_DEV int pick_start(double en, double ep)
{
    if (ep <= en && ep <= 0.0) return 0;
    return en <= 0.0 ? 1 : 2;
}

// x0 holds v_prev on entry
__global__ void k_pick(int64_t len, const double *s_net, const double *s_prev, const double *guess, double *x0)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= len) return;
    const double en = 0.5 * s_net[0] - s_net[1], ep = 0.5 * s_prev[0] - s_prev[1];
    const int k = pick_start(en, ep);
    if (k == 1) x0[t] = guess[t];
    if (k == 2) x0[t] = 0.0;
}

__global__ void k_sum_double(const double *part, int np, double *out)
{
    __shared__ double sh[256];
    double s = 0.0;
    for (int k = threadIdx.x; k < np; k += 256) s += part[k];
    s = block_sum_256(s, sh);
    if (threadIdx.x == 0) *out = s;
}

__global__ void k_output(int64_t n, const int32_t *perm, const float *out16, const float *bout, double sV,
                         double *vhat)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    for (int a = 0; a < 3; a++) vhat[3 * u + a] = sV * (double)(out16[16 * i + a] + bout[a]);
}

__global__ void k_adam(int64_t np, float *theta, const float *g, float *m1, float *m2, float lr, float b1, float b2,
                       float eps, float c1, float c2)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= np) return;
    float gt = g[t];
    float a = b1 * m1[t] + (1.f - b1) * gt;
    float b = b2 * m2[t] + (1.f - b2) * gt * gt;
    m1[t] = a;
    m2[t] = b;
    theta[t] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// ---------------------------------------------------------------- host drivers

struct Act {
    float *x16, *pre0, *h[NL + 1], *PQ, *a[NL], *U[NL], *out16;   // forward
    float *dout16, *dh, *dU, *dcat, *dPQ, *tmp;                    // backward
};

int64_t act_floats(int64_t n) { return n * (16 + 64 + 64 * (NL + 1) + 128 + 64 * NL + 64 * NL + 16 + 16 + 64 + 64 + 128 + 128 + 64); }

Act carve(float *base, int64_t n)
{
    Act A;
    float *p = base;
    auto take = [&](int64_t cnt) { float *q = p; p += cnt; return q; };
    A.x16 = take(16 * n);
    A.pre0 = take(64 * n);
    for (int l = 0; l <= NL; l++) A.h[l] = take(64 * n);
    A.PQ = take(128 * n);
    for (int l = 0; l < NL; l++) A.a[l] = take(64 * n);
    for (int l = 0; l < NL; l++) A.U[l] = take(64 * n);
    A.out16 = take(16 * n);
    A.dout16 = take(16 * n);
    A.dh = take(64 * n);
    A.dU = take(64 * n);
    A.dcat = take(128 * n);
    A.dPQ = take(128 * n);
    A.tmp = take(64 * n);
    return A;
}

int gemm(sgp_ctx ctx, const float *A, int64_t lda, const unsigned short *B, float *C, int64_t ldc, int64_t M, int K,
         int N, const float *bias, float *relu_out = nullptr)
{
    if (M <= 0) return SGP_OK;
    const int64_t nb = grid_for(M, GEMM_ROWS);
    hipStream_t st = ctx->stream;
    float *R = relu_out;
    switch (K) {
    case 16: k_gemm<1, false><<<nb, 256, 0, st>>>(A, lda, B, C, ldc, M, N, bias, R, {}); break;
    case 64: k_gemm<4, false><<<nb, 256, 0, st>>>(A, lda, B, C, ldc, M, N, bias, R, {}); break;
    default: return set_err(ctx, SGP_EINVAL, "mpnn gemm: unsupported K");
    }
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

// a product of the backward pass with N = 64 (GemmBack)
template <int KT>
int gemm_back(sgp_ctx ctx, const float *A, const unsigned short *B, float *C, int64_t M, const GemmBack &bk)
{
    if (M <= 0) return SGP_OK;
    k_gemm<KT, true><<<grid_for(M, GEMM_ROWS), 256, 0, ctx->stream>>>(A, 16 * KT, B, C, 64, M, 64, nullptr, nullptr, bk);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

// the fixed-order sum of the G partial vectors part[g][0, L), into the gradient
int reduce_parts(sgp_ctx ctx, const float *part, int G, int L, const GradOut &o)
{
    k_red_out<<<grid_for(L, 64), 64 * RED_WAVES, 0, ctx->stream>>>(part, G, L, o);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

// [A | A2]^T D (16 (KT1 + KT2) x 16 NT) and the column sums of D over all m
// rows, into the gradient
template <int KT1, int KT2, int NT>
int gemm_at(sgp_ctx ctx, sgp_mpnn M, const float *A, int64_t lda, const float *A2, int64_t lda2, const float *D,
            int64_t ldd, int64_t m, GradOut o)
{
    constexpr int K = 16 * (KT1 + KT2), N = 16 * NT, L = K * N + N;
    const int G = (int)std::min<int64_t>(std::max<int64_t>((m + 63) / 64, 1), AT_GRID);
    float *part;
    SGP_TRY(ensure_t(ctx, M->part, (size_t)G * L + 64, &part));
    k_gemm_at<KT1, KT2, NT><<<G, 256, 0, ctx->stream>>>(A, lda, A2, lda2, D, ldd, m, part);
    LAUNCH_CHECK(ctx);
    o.K = K;
    o.N = N;
    return reduce_parts(ctx, part, G, L, o);
}

int prepare(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, const double *F, const double *vp, Act &A)
{
    const int64_t n = g->n, ne = 2 * g->m;
    float *base;
    float4 *ef;
    int32_t *irow, *icol, *deg;
    SGP_TRY(ensure_t(ctx, M->act, (size_t)act_floats(n) + 64, &base));
    SGP_TRY(ensure_t(ctx, M->efeat, (size_t)ne + 1, &ef));
    SGP_TRY(ensure_t(ctx, M->irow, (size_t)n + 2, &irow));
    SGP_TRY(ensure_t(ctx, M->icol, (size_t)ne + 1, &icol));
    SGP_TRY(ensure_t(ctx, ctx->ws[WS_DEG], (size_t)n + 2, &deg));
    A = carve(base, n);
    hipStream_t st = ctx->stream;
    const int32_t *perm = (const int32_t *)g->perm.p;
    k_input<<<grid_for(n, 256), 256, 0, st>>>(n, perm, F, vp, (float)M->sF, (float)M->sV, A.x16);
    LAUNCH_CHECK(ctx);
    // the internal neighbour lists depend only on the graph and sW: rebuilt
    // when either changed since the last call
    if (M->lists_of != g || M->lists_version != g->version || M->lists_sW != M->sW) {
        k_int_deg<<<grid_for(n, 256), 256, 0, st>>>(n, perm, (const int32_t *)g->rowptr.p, deg);
        LAUNCH_CHECK(ctx);
        SGP_TRY(scan_exclusive(ctx, deg, irow, n));
        k_int_entries<<<grid_for(16 * n, 256), 256, 0, st>>>(n, perm, (const int32_t *)g->inv.p,
                                                             (const int32_t *)g->rowptr.p, (const int32_t *)g->col.p,
                                                             (const int32_t *)g->ent_edge.p, (const double4 *)g->wu.p,
                                                             (float)M->sW, irow, icol, ef);
        LAUNCH_CHECK(ctx);
        M->lists_of = g;
        M->lists_version = g->version;
        M->lists_sW = M->sW;
    }
    return SGP_OK;
}

// keep: pre0 and U of every layer are kept for a backward pass
int forward(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, Act &A, bool keep)
{
    hipStream_t st = ctx->stream;
    const int64_t n = g->n;
    const unsigned short *W = (const unsigned short *)M->wbf.p;
    const float *wr = (const float *)M->wrow.p;
    const Layout &L = M->L;
    const Packed &PK = M->PK;
    const int32_t *rowptr = (const int32_t *)M->irow.p, *col = (const int32_t *)M->icol.p;   // internal order
    const float4 *ef = (const float4 *)M->efeat.p;
    // input layer: pre0 kept for the backward pass, h0 = relu(pre0) in the same pass
    SGP_TRY(gemm(ctx, A.x16, 16, W + PK.in16, A.pre0, 64, n, 16, 64, wr + L.b_in, A.h[0]));
    SGP_TRY(gemm(ctx, A.h[0], 64, W + PK.ab[0], A.PQ, 128, n, 64, 128, nullptr));
    // the layers gather from one PQ and write the next one's to the other
    // buffer (dPQ, free in a forward pass); the last layer's is in PQ
    static_assert(NL % 2 == 1, "the last layer reads A.PQ");
    const bf16x4 *B = (const bf16x4 *)M->wfrag.p;
    const unsigned grid = (unsigned)((n + LAYER_ROWS - 1) / LAYER_ROWS);
    for (int l = 0; l < NL && n > 0; l++, B += FRAG_LAYER) {
        float *agg = keep ? A.a[l] : nullptr, *U = keep ? A.U[l] : nullptr;
        const float *PQ = l % 2 ? A.dPQ : A.PQ;
        if (l < NL - 1)
            k_layer<8><<<grid, 256, 0, st>>>(n, rowptr, col, ef, PQ, wr + L.b_m[l], wr + L.W_c[l], A.h[l], B,
                                             wr + L.b_u[l], B + FRAG_U, agg, U, A.h[l + 1], l % 2 ? A.PQ : A.dPQ, 128);
        else   // (b_out is added where the output is read: k_output, k_loss)
            k_layer<1><<<grid, 256, 0, st>>>(n, rowptr, col, ef, PQ, wr + L.b_m[l], wr + L.W_c[l], A.h[l], B,
                                             wr + L.b_u[l], B + FRAG_U, agg, U, keep ? A.h[l + 1] : nullptr, A.out16,
                                             16);
    }
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

int backward(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, Act &A)
{
    hipStream_t st = ctx->stream;
    const int64_t n = g->n;
    const unsigned short *W = (const unsigned short *)M->wbf.p;
    const float *wr = (const float *)M->wrow.p;
    const Layout &L = M->L;
    const Packed &PK = M->PK;
    float *G = (float *)M->grad.p;
    const int32_t *rowptr = (const int32_t *)M->irow.p, *col = (const int32_t *)M->icol.p;   // internal order
    const float4 *ef = (const float4 *)M->efeat.p;
    // output layer: W_out rows 0..63 x columns 0..2 of h^T dout, b_out = column sums
    SGP_TRY((gemm_at<4, 0, 1>(ctx, M, A.h[NL], 64, nullptr, 0, A.dout16, 16, n,
                              {G + L.W_out, nullptr, G + L.b_out, 0, 0, 64, 3, 3, 3})));
    // dh of the last layer's output, and dU = dh where U > 0
    SGP_TRY(gemm_back<1>(ctx, A.dout16, W + PK.out16T, A.dh, n, {nullptr, nullptr, 0, A.U[NL - 1], A.dU}));
    for (int l = NL - 1; l >= 0; l--) {
        // W_u = [h | a]^T dU, b_u = column sums of dU
        SGP_TRY((gemm_at<4, 4, 4>(ctx, M, A.h[l], 64, A.a[l], 64, A.dU, 64, n,
                                  {G + L.W_u[l], nullptr, G + L.b_u[l], 0, 0, 128, 64, 64, 64})));
        SGP_TRY(gemm(ctx, A.dU, 64, W + PK.uT[l], A.dcat, 128, n, 64, 128, nullptr));   // [dh part | da]
        // messages: recompute PQ of this layer from h[l] (the last layer's is
        // still there from the forward pass)
        if (l < NL - 1) SGP_TRY(gemm(ctx, A.h[l], 64, W + PK.ab[l], A.PQ, 128, n, 64, 128, nullptr));
        const int nb = (int)std::min<int64_t>(grid_for(n, 16), MSG_BWD_GRID);
        float *wcp;
        SGP_TRY(ensure_t(ctx, ctx->ws[WS_TMP9], (size_t)nb * 256 + 64, &wcp));
        k_msg_bwd_p<<<nb, 256, 0, st>>>(n, rowptr, col, ef, A.PQ, wr + L.b_m[l], wr + L.W_c[l], A.dcat + 64, 128,
                                        A.dPQ, wcp);
        k_msg_bwd_q<<<grid_for(n, 16), 256, 0, st>>>(n, rowptr, col, ef, A.PQ, wr + L.b_m[l], wr + L.W_c[l],
                                                     A.dcat + 64, 128, A.dPQ);
        LAUNCH_CHECK(ctx);
        SGP_TRY(reduce_parts(ctx, wcp, nb, 256, {G + L.W_c[l], nullptr, nullptr, 4, 64, 4, 64, 64, 64}));   // 4 x 64
        // W_a, W_b = h^T dP, h^T dQ; b_m = column sums of dP
        SGP_TRY((gemm_at<4, 0, 8>(ctx, M, A.h[l], 64, nullptr, 0, A.dPQ, 128, n,
                                  {G + L.W_a[l], G + L.W_b[l], G + L.b_m[l], 0, 0, 64, 64, 128, 64})));
        // dh_l = dh (residual) + dcat[:, :64] + dPQ W_ab^T, and its part where
        // the activation before it passed (the input layer's for l = 0)
        SGP_TRY(gemm_back<8>(ctx, A.dPQ, W + PK.abT[l], l > 0 ? A.tmp : nullptr, n,
                             {A.dh, A.dcat, 128, l > 0 ? A.U[l - 1] : A.pre0, A.dU}));
        std::swap(A.dh, A.tmp);
    }
    SGP_TRY((gemm_at<1, 0, 4>(ctx, M, A.x16, 16, nullptr, 0, A.dU, 64, n,
                              {G + L.W_in, nullptr, G + L.b_in, 0, 0, 6, 64, 64, 64})));
    return SGP_OK;
}

int repack(sgp_ctx ctx, sgp_mpnn M)
{
    unsigned short *wbf;
    float *wr;
    SGP_TRY(ensure_t(ctx, M->wbf, (size_t)M->PK.total + 8, &wbf));
    SGP_TRY(ensure_t(ctx, M->wrow, (size_t)M->L.total + 8, &wr));
    int64_t cnt = std::max<int64_t>(M->PK.total, M->L.total);
    k_pack<<<grid_for(cnt, 256), 256, 0, ctx->stream>>>((const float *)M->theta.p, M->L, M->PK, wbf, wr);
    bf16x4 *fr;
    SGP_TRY(ensure_t(ctx, M->wfrag, (size_t)NL * FRAG_LAYER, &fr));
    k_pack_frag<<<grid_for(NL * FRAG_LAYER, 256), 256, 0, ctx->stream>>>(wbf, M->PK, fr);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

}   // namespace

// ---------------------------------------------------------------- C ABI

extern "C" int sgp_mpnn_param_count(int64_t *count)
{
    if (!count) return SGP_EINVAL;
    *count = make_layout().total;
    return SGP_OK;
}

extern "C" int sgp_mpnn_create(sgp_ctx ctx, sgp_mpnn *out)
{
    if (!ctx || !out) return set_err(ctx, SGP_EINVAL, "mpnn_create: null");
    *out = new (std::nothrow) sgp_mpnn_();
    return *out ? SGP_OK : set_err(ctx, SGP_ENOMEM, "mpnn_create: out of memory");
}

extern "C" void sgp_mpnn_free(sgp_mpnn M)
{
    if (!M) return;
    (void)hipDeviceSynchronize();
    release(M->theta); release(M->m1); release(M->m2); release(M->grad); release(M->wbf); release(M->wfrag); release(M->wrow);
    release(M->act); release(M->efeat); release(M->part); release(M->vq);
    release(M->irow); release(M->icol);
    delete M;
}

extern "C" int sgp_mpnn_set_params(sgp_ctx ctx, sgp_mpnn M, const float *theta, double sF, double sV, double sW)
{
    if (!ctx || !M || !theta || !(sF > 0) || !(sV > 0) || !(sW > 0))
        return set_err(ctx, SGP_EINVAL, "mpnn_set_params: bad arguments");
    const int64_t np = M->L.total;
    float *t, *a, *b, *gr;
    SGP_TRY(ensure_t(ctx, M->theta, np + 8, &t));
    SGP_TRY(ensure_t(ctx, M->m1, np + 8, &a));
    SGP_TRY(ensure_t(ctx, M->m2, np + 8, &b));
    SGP_TRY(ensure_t(ctx, M->grad, np + 8, &gr));
    HIP_TRY(ctx, hipMemcpyAsync(t, theta, np * sizeof(float), hipMemcpyDeviceToDevice, ctx->stream));
    HIP_TRY(ctx, hipMemsetAsync(a, 0, np * sizeof(float), ctx->stream));
    HIP_TRY(ctx, hipMemsetAsync(b, 0, np * sizeof(float), ctx->stream));
    M->sF = sF;
    M->sV = sV;
    M->sW = sW;
    M->adam_t = 0;
    return repack(ctx, M);
}

extern "C" int sgp_mpnn_get_params(sgp_ctx ctx, sgp_mpnn M, float *theta)
{
    if (!ctx || !M || !theta || !M->theta.p) return set_err(ctx, SGP_EINVAL, "mpnn_get_params: bad arguments");
    HIP_TRY(ctx, hipMemcpyAsync(theta, M->theta.p, M->L.total * sizeof(float), hipMemcpyDeviceToDevice, ctx->stream));
    return SGP_OK;
}

static int check_common(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, const double *F, const double *vp)
{
    if (!ctx || !M || !g || !M->theta.p) return set_err(ctx, SGP_EINVAL, "mpnn: missing handle or parameters");
    if (g->n > 0 && (!F || !vp)) return set_err(ctx, SGP_EINVAL, "mpnn: null input");
    return SGP_OK;
}

extern "C" int sgp_mpnn_forward(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, const double *F, const double *vprev,
                                double *vhat)
{
    SGP_TRY(check_common(ctx, M, g, F, vprev));
    if (g->n == 0) return SGP_OK;
    if (!vhat) return set_err(ctx, SGP_EINVAL, "mpnn_forward: null output");
    Act A;
    SGP_TRY(prepare(ctx, M, g, F, vprev, A));
    SGP_TRY(forward(ctx, M, g, A, false));
    k_output<<<grid_for(g->n, 256), 256, 0, ctx->stream>>>(g->n, (const int32_t *)g->perm.p, A.out16,
                                                            (const float *)M->wrow.p + M->L.b_out, M->sV, vhat);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

// sums (x . Gamma x, x . F, v . F) of a canonical-order x into s[0..2]; q
// receives Gamma x.  Uses the library's product (workspaces of sgp_spmv).
static int energy_sums(sgp_ctx ctx, sgp_mpnn M, sgp_bsr A, const double *x, double *q, const double *F,
                       const double *v, double *s)
{
    const int64_t n = A->n;
    SGP_TRY(sgp_spmv(ctx, A, x, q));
    const int nb = (int)std::min<int64_t>(grid_for(3 * n, 256), 1024);
    double *part;
    SGP_TRY(ensure_t(ctx, ctx->ws[WS_PART], (size_t)3 * nb + 8, &part));
    k_energy_parts<<<nb, 256, 0, ctx->stream>>>(3 * n, x, q, F, v, part);
    k_sum3<<<1, 256, 0, ctx->stream>>>(part, nb, s);
    LAUNCH_CHECK(ctx);
    return SGP_OK;
}

static int loss_grad(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, sgp_bsr Gm, const double *F, const double *vprev,
                     const double *v, double *loss)
{
    Act A;
    const int64_t n = g->n;
    SGP_TRY(prepare(ctx, M, g, F, vprev, A));
    SGP_TRY(forward(ctx, M, g, A, true));
    double s[3];
    if (!Gm) {
        double *part;
        const int nb = (int)grid_for(n, 256);
        SGP_TRY(ensure_t(ctx, ctx->ws[WS_PART], (size_t)nb + 8, &part));
        k_loss<<<nb, 256, 0, ctx->stream>>>(n, (const int32_t *)g->perm.p, A.out16,
                                            (const float *)M->wrow.p + M->L.b_out, v, (float)M->sV, A.dout16, part);
        k_sum_double<<<1, 256, 0, ctx->stream>>>(part, nb, part + nb);
        LAUNCH_CHECK(ctx);
        SGP_TRY(backward(ctx, M, g, A));
        SGP_TRY(readback(ctx, s, part + nb, sizeof(double)));
        if (loss) *loss = s[0] / (3.0 * (double)n);
        return SGP_OK;
    }
    // energy loss (v_hat' G v_hat - 2 v_hat' F + v' F) / (v' F)
    double *vh, *ds;
    SGP_TRY(ensure_t(ctx, M->vq, (size_t)6 * n + 8, &vh));
    double *q = vh + 3 * n, *sd = vh + 6 * n;
    ds = sd;
    k_output<<<grid_for(n, 256), 256, 0, ctx->stream>>>(n, (const int32_t *)g->perm.p, A.out16,
                                                      (const float *)M->wrow.p + M->L.b_out, M->sV, vh);
    LAUNCH_CHECK(ctx);
    SGP_TRY(energy_sums(ctx, M, Gm, vh, q, F, v, ds));
    k_energy_dout<<<grid_for(n, 256), 256, 0, ctx->stream>>>(n, (const int32_t *)g->perm.p, q, F, M->sV, ds,
                                                            A.dout16);
    LAUNCH_CHECK(ctx);
    SGP_TRY(backward(ctx, M, g, A));
    SGP_TRY(readback(ctx, s, ds, sizeof s));
    if (loss) *loss = (s[0] - 2.0 * s[1] + s[2]) / s[2];
    return SGP_OK;
}

static int check_gamma(sgp_ctx ctx, sgp_graph g, sgp_bsr Gm)
{
    if (Gm && Gm->n != g->n) return set_err(ctx, SGP_EINVAL, "mpnn: Gamma and graph sizes differ");
    return SGP_OK;
}

extern "C" int sgp_mpnn_grad(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, sgp_bsr Gm, const double *F, const double *vprev,
                             const double *v, float *grad, double *loss)
{
    SGP_TRY(check_common(ctx, M, g, F, vprev));
    if (!v || !grad || g->n == 0) return set_err(ctx, SGP_EINVAL, "mpnn_grad: bad arguments");
    SGP_TRY(check_gamma(ctx, g, Gm));
    SGP_TRY(loss_grad(ctx, M, g, Gm, F, vprev, v, loss));
    HIP_TRY(ctx, hipMemcpyAsync(grad, M->grad.p, M->L.total * sizeof(float), hipMemcpyDeviceToDevice, ctx->stream));
    return SGP_OK;
}

extern "C" int sgp_mpnn_train_step(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, sgp_bsr Gm, const double *F,
                                   const double *vprev, const double *v, double lr, double *loss)
{
    SGP_TRY(check_common(ctx, M, g, F, vprev));
    if (!v || g->n == 0 || !(lr > 0)) return set_err(ctx, SGP_EINVAL, "mpnn_train_step: bad arguments");
    SGP_TRY(check_gamma(ctx, g, Gm));
    SGP_TRY(loss_grad(ctx, M, g, Gm, F, vprev, v, loss));
    M->adam_t++;
    const float b1 = 0.9f, b2 = 0.999f;
    float c1 = 1.f - powf(b1, (float)M->adam_t), c2 = 1.f - powf(b2, (float)M->adam_t);
    k_adam<<<grid_for(M->L.total, 256), 256, 0, ctx->stream>>>(M->L.total, (float *)M->theta.p, (const float *)M->grad.p,
                                                              (float *)M->m1.p, (float *)M->m2.p, (float)lr, b1, b2,
                                                              1e-8f, c1, c2);
    LAUNCH_CHECK(ctx);
    return repack(ctx, M);
}

extern "C" int sgp_mpnn_warm_start(sgp_ctx ctx, sgp_mpnn M, sgp_graph g, sgp_bsr Gm, const double *F,
                                   const double *vprev, double *x0, int32_t *used_net, double *energy_net,
                                   double *energy_prev)
{
    SGP_TRY(check_common(ctx, M, g, F, vprev));
    if (!Gm || (g->n > 0 && !x0)) return set_err(ctx, SGP_EINVAL, "mpnn_warm_start: bad arguments");
    SGP_TRY(check_gamma(ctx, g, Gm));
    const int64_t n = g->n;
    if (n == 0) {
        if (used_net) *used_net = 0;
        if (energy_net) *energy_net = 0.0;
        if (energy_prev) *energy_prev = 0.0;
        return SGP_OK;
    }
    Act A;
    SGP_TRY(prepare(ctx, M, g, F, vprev, A));
    SGP_TRY(forward(ctx, M, g, A, false));
    double *vh;
    SGP_TRY(ensure_t(ctx, M->vq, (size_t)6 * n + 8, &vh));
    double *q = vh + 3 * n, *s = vh + 6 * n;   // s: 3 sums of the guess, 3 of v_prev (8 doubles reserved)
    k_output<<<grid_for(n, 256), 256, 0, ctx->stream>>>(n, (const int32_t *)g->perm.p, A.out16,
                                                      (const float *)M->wrow.p + M->L.b_out, M->sV, vh);
    LAUNCH_CHECK(ctx);
    SGP_TRY(energy_sums(ctx, M, Gm, vh, q, F, nullptr, s));
    SGP_TRY(energy_sums(ctx, M, Gm, vprev, q, F, nullptr, s + 3));
    if (x0 != vprev)
        HIP_TRY(ctx, hipMemcpyAsync(x0, vprev, 3 * n * sizeof(double), hipMemcpyDeviceToDevice, ctx->stream));
    k_pick<<<grid_for(3 * n, 256), 256, 0, ctx->stream>>>(3 * n, s, s + 3, vh, x0);
    LAUNCH_CHECK(ctx);
    double hs[6];
    SGP_TRY(readback(ctx, hs, s, sizeof hs));
    const double en = 0.5 * hs[0] - hs[1], ep = 0.5 * hs[3] - hs[4];
    // the host's choice repeats the kernel's comparisons on the same values
    if (used_net) *used_net = (ep <= en && ep <= 0.0) ? 0 : (en <= 0.0 ? 1 : 2);
    if (energy_net) *energy_net = en;
    if (energy_prev) *energy_prev = ep;
    return SGP_OK;
}
