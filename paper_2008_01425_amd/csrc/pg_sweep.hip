// Edge sweeps: both products of a power step in one pass over the parameters.
//
// With D = X_a - X_b the power step of an edge is P = D Q, Phat = P R^-1 (Gram-Schmidt), Q' = D^T Phat = (D^T P) R^-1.
// A work-group takes a block of rows of BOTH workers of an edge: it forms P for those rows and, while they are in
// registers, adds their share of D^T P.  Only R, a handful of numbers per (edge, layer), needs all rows, and it is applied
// afterwards to the vectors (sweep_finish_kernel).  So a step reads the parameters once where the products worker by worker read
// them twice with the orthonormalisation between.
//
// A worker's rows are wanted by each of its edges.  The work-groups of one block of rows, all edges, run on one die
// (every eighth work-group goes to the same one) next to each other, so that its L2 serves all but the first: one matrix of
// 2048 x 4608 on 16 workers, ring, 604 MB: 111 us, 5.4 TB/s of parameters read once (a plain read pass takes 101 us); with
// the edges spread over the dies 163 us.
//
// Measured, streaming kernels -> sweeps: VGG-16 shapes, ring of 16, SGD round 812 -> 735 us (this kernel 225 us for 0.94 GB, issue of a row's chain and
// HBM about even); ResNet-20 shapes, ring of 8, SGD round 29.8 -> 23.9 us; eight layers of odd lengths on a tree of 11 at rank 3 466 -> 249 us, with the update in one launch.
#include "pg_device.h"
#include "pg_launch.h"

namespace pg {

__device__ __forceinline__ double row16_sum(double z) {
    z += dpp_mov<0xB1>(z);
    z += dpp_mov<0x4E>(z);
    z += dpp_mov<0x141>(z);
    z += dpp_mov<0x140>(z);
    return z;
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// N values summed over the wavefront; every lane receives all sums (as scalars)
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N]) {
#pragma unroll
    for (int i = 0; i + 4 <= N; i += 4) {
        const double z = row16_sum(fold16(fold32(v[i], v[i + 2]), fold32(v[i + 1], v[i + 3])));
#pragma unroll
        for (int k = 0; k < 4; ++k) v[i + k] = read_lane(z, 16 * k);
    }
    if constexpr (N % 4 >= 2) {
        constexpr int i = N / 4 * 4;
        const double f = fold32(v[i], v[i + 1]);
        const double z = row16_sum(fold16(f, f));
        v[i] = read_lane(z, 0);
        v[i + 1] = read_lane(z, 32);
    }
    if constexpr (N % 2 == 1) {
        const double f = fold32(v[N - 1], v[N - 1]);
        const double z = row16_sum(fold16(f, f));
        v[N - 1] = read_lane(z, 0);
    }
}

template <int I>
struct IntTag {
    static constexpr int value = I;
};
// Entry i of the packed Gram matrix (j <= k at k (k + 1) / 2 + j) of columns that are orthonormal, or dropped and zero.
__device__ __forceinline__ double sweep_unit_gram(int i, const int *drop) {
    int k = 0;
    while ((k + 1) * (k + 2) / 2 <= i) ++k;
    return i == k * (k + 1) / 2 + k && !drop[k] ? 1.0 : 0.0;
}

// One tile: rows [row0, row0 + nrows) of one (edge, layer).
//   TC = 2^tc_shift threads side by side over the units (four floats) of a row, K units each; NT / TC groups of threads take
//   M rows each per step, B steps ahead in registers.  A row's last unit, if it reaches past the end, is moved back to the last four
//   floats; the ones its neighbour owns, and the units of threads past the end, meet zeros in the right vectors and
//   their column sums are not stored.  q >= 4.
//   EXACT (small layers, one block): the rows are walked twice, the second time with Phat as it is stored, rounded to float.  A layer of
//   a few hundred entries loses its difference within a few rounds, and the last bits of Phat decide what the next ones see.
// Bound by HBM where a row block's workers share an L2, by instruction issue where each row is wanted by four edges.
template <int NT, int RM, int K, int M, int B, bool EXACT>
__device__ __forceinline__ void sweep_body(const SweepTile &t, const SweepDesc &d, const float *Xa, const float *Xb, const float *__restrict__ qin,
                                           double *__restrict__ part, char *lds) {
    constexpr int NG = RM * (RM + 1) / 2;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = d.q, r = RM == 1 ? 1 : d.r;
    const int TC = 1 << d.tc_shift, G = NT >> d.tc_shift;
    const int tc = tid & (TC - 1), g = TC >= 64 ? wave >> (d.tc_shift - 6) : tid >> d.tc_shift;
    const int nv = (q + 3) >> 2, vs = 4 * K * TC;
    const int last = q - 4, row_end = t.row0 + t.nrows;
    const int wc = TC > 64 ? TC >> 6 : 1;  // wavefronts that share a row

    float *sV = reinterpret_cast<float *>(lds);                       // [r][vs]: right vectors, unit by unit
    double *sPart = reinterpret_cast<double *>(lds + r * vs * 4);     // [2][wavefronts][M * RM]: row sums of the wavefronts
    double *sP = sPart + 2 * (NT / 64) * M * RM;                      // EXACT: [r][nrows] P, then Phat
    __shared__ double sGram[NT / 64][NG], sG[NG], sR[RM][RM];
    __shared__ int sDrop[RM];
    // float i of a vector laid out unit by unit: column i, those of the last unit moved back
    auto slot = [&](int i) { return i < 4 * (nv - 1) ? i : i < 4 * nv ? last + (i & 3) : q; };
    uint32_t col[K];  // byte offsets of this thread's units in a row
#pragma unroll
    for (int k = 0; k < K; ++k) col[k] = 4u * (uint32_t)min(4 * (tc + k * TC), last);

    double acc[RM][K][4], gram[NG];
#pragma unroll
    for (int j = 0; j < RM; ++j)
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[j][k][v] = 0.0;
#pragma unroll
    for (int i = 0; i < NG; ++i) gram[i] = 0.0;

    struct Buf {
        float a[M][K][4], b[M][K][4];
    };
    auto load = [&](int row, Buf &x) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const uint32_t at = 4u * (uint32_t)min(row + m, row_end - 1) * (uint32_t)d.ld;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                ld4_at(Xa, at + col[k], x.a[m][k]);
                ld4_at(Xb, at + col[k], x.b[m][k]);
            }
        }
    };
    const int step_rows = G * M;
    Buf x[B];
    auto prime = [&]() {
#pragma unroll
        for (int i = 0; i < B; ++i) load(t.row0 + (i * G + g) * M, x[i]);
    };
    prime();
    // the right vectors, several loads at a time, behind the first rows
    constexpr int S = 4;
    for (int i0 = tid; i0 < r * vs; i0 += S * NT) {
        float y[S];
        bool own[S];
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int at = min(i0 + u * NT, r * vs - 1), k = RM == 1 ? 0 : at / vs, i = at - k * vs, c = slot(i);
            own[u] = c < q && (i < 4 * (nv - 1) || c >= 4 * (nv - 1));
            y[u] = ldg1(qin + d.q_off + (int64_t)k * q + min(c, q - 1));
        }
#pragma unroll
        for (int u = 0; u < S; ++u)
            if (i0 + u * NT < r * vs) sV[i0 + u * NT] = own[u] ? y[u] : 0.0f;
    }
    const int steps = (t.nrows + step_rows - 1) / step_rows;
    auto gram_sum = [&]() {  // over the groups of a wavefront, then over the wavefronts (those of one row hold copies)
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            for (int x = TC; x < 64; x <<= 1) gram[i] += __shfl_xor(gram[i], x);
            if (lane == 0) sGram[wave][i] = gram[i];
        }
        __syncthreads();
        if (tid < NG) {
            double sum = 0.0;
            for (int w = 0; w < NT / 64; w += wc) sum += sGram[w][tid];
            sG[tid] = sum;
        }
        __syncthreads();
    };
    // PHASE 0: P, its Gram sums and (not EXACT) the column sums with it; 1: the column sums with the rounded Phat
    auto step = [&](auto phase, int s, Buf &x) {
        constexpr int PHASE = decltype(phase)::value;
        const int row = t.row0 + (s * G + g) * M;
        double D[M][K][4];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int v = 0; v < 4; ++v) D[m][k][v] = (double)x.a[m][k][v] - (double)x.b[m][k][v];
        PG_FENCE();
        load(row + B * step_rows, x);  // (past the block's end: its last row again)
        PG_FENCE();
        double p[M * RM];
        if constexpr (PHASE == 0) {
#pragma unroll
            for (int i = 0; i < M * RM; ++i) p[i] = 0.0;
#pragma unroll
            for (int j = 0; j < RM; ++j) {
                if (j >= r) continue;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const VecT<4>::T w = *reinterpret_cast<const VecT<4>::T *>(sV + j * vs + 4 * (tc + k * TC));
#pragma unroll
                    for (int m = 0; m < M; ++m)
#pragma unroll
                        for (int v = 0; v < 4; ++v) p[m * RM + j] = fma(D[m][k][v], (double)w[v], p[m * RM + j]);
                }
            }
            // An infinite parameter in a float that is not this thread's own met a zero: without that float.  (A test per step; a mask on
            // every float would be two instructions more for each.)
            bool nan = false;
#pragma unroll
            for (int i = 0; i < M * RM; ++i) nan = nan || p[i] != p[i];
            if (nan && 4 * (tc + (K - 1) * TC) > last) {
                int at = 4 * tc;
                asm volatile("" : "+v"(at));  // (empty: keeps the masks from being formed, and held, ahead of the loop)
#pragma unroll
                for (int j = 0; j < RM; ++j) {
                    if (j >= r) continue;
#pragma unroll
                    for (int m = 0; m < M; ++m) p[m * RM + j] = 0.0;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const VecT<4>::T w = *reinterpret_cast<const VecT<4>::T *>(sV + j * vs + at + 4 * k * TC);
                        const int back = at + 4 * k * TC - last;  // floats of the unit that are not its own (none: 0 or less)
#pragma unroll
                        for (int m = 0; m < M; ++m)
#pragma unroll
                            for (int v = 0; v < 4; ++v) p[m * RM + j] = fma(v < back ? 0.0 : D[m][k][v], (double)w[v], p[m * RM + j]);
                    }
                }
            }
            if (TC < 64) {
                group_sum_all<M * RM>(p, TC);
            } else {
                wave_sums<M * RM>(p);
                if (TC > 64) {
                    double *mine = sPart + ((s & 1) * (NT / 64) + wave) * (M * RM);
                    if (lane == 0) {
#pragma unroll
                        for (int i = 0; i < M * RM; ++i) mine[i] = p[i];
                    }
                    __syncthreads();
                    const double *all = sPart + ((s & 1) * (NT / 64) + (wave & ~(wc - 1))) * (M * RM);
#pragma unroll
                    for (int i = 0; i < M * RM; ++i) p[i] = all[i];
                    for (int w = 1; w < wc; ++w)
#pragma unroll
                        for (int i = 0; i < M * RM; ++i) p[i] += all[w * (M * RM) + i];
                }
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const bool ok = row + m < row_end;
#pragma unroll
                for (int j = 0; j < RM; ++j) {
                    if (ok && tc == 0 && j < r) {
                        if (EXACT) sP[j * t.nrows + row + m - t.row0] = p[m * RM + j];
                        else part[d.pe_off + (int64_t)j * d.p + row + m] = p[m * RM + j];
                    }
                    p[m * RM + j] = ok ? p[m * RM + j] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < RM; ++j)
#pragma unroll
                    for (int i = 0; i <= j; ++i) gram[j * (j + 1) / 2 + i] = fma(p[m * RM + i], p[m * RM + j], gram[j * (j + 1) / 2 + i]);
            }
        } else {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int j = 0; j < RM; ++j)
                    p[m * RM + j] = row + m < row_end && j < r ? sP[j * t.nrows + row + m - t.row0] : 0.0;
        }
        if constexpr (!EXACT || PHASE == 1) {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int j = 0; j < RM; ++j)
#pragma unroll
                    for (int k = 0; k < K; ++k)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[j][k][v] = fma(D[m][k][v], p[m * RM + j], acc[j][k][v]);
        }
        PG_FENCE();
    };
    auto walk = [&](auto phase) {
        __syncthreads();  // vectors staged; P complete
        for (int s = 0; s < steps; s += B) {  // (a step past the block's end adds nothing; skipping it would make every wait a full one)
#pragma unroll
            for (int i = 0; i < B; ++i) step(phase, s + i, x[i]);
        }
    };
    walk(IntTag<0>());
    gram_sum();
    if constexpr (EXACT) {
        prime();
        gram_factor<RM>(r, sG, sR, sDrop, nullptr);
        for (int i = tid; i < t.nrows; i += NT) {
            double ph[RM];
#pragma unroll
            for (int k = 0; k < RM; ++k) {
                ph[k] = 0.0;
                if (k >= r) continue;
                double v = sP[k * t.nrows + i];
#pragma unroll
                for (int j = 0; j < k; ++j) v -= sR[j][k] * ph[j];
                ph[k] = sDrop[k] ? 0.0 : v / sR[k][k];
                sP[k * t.nrows + i] = (double)(float)ph[k];
                part[d.pe_off + (int64_t)k * d.p + t.row0 + i] = (double)(float)ph[k];
            }
        }
        walk(IntTag<1>());
        __syncthreads();
    }

    // this block's column sums: lanes and groups that hold other rows of the same columns, through LDS, in a fixed order
    double *red = reinterpret_cast<double *>(lds);
    double *dst = part + d.qe_off + (int64_t)t.blk * r * q;
    const int groups = TC >= 64 ? G : NT / 64;  // wavefronts with the same columns
#pragma unroll
    for (int j = 0; j < RM; ++j) {
        if (j >= r) continue;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            for (int x = TC; x < 64; x <<= 1)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[j][k][v] += __shfl_xor(acc[j][k][v], x);
            if (groups == 1) {  // every column is one thread's
                const int c = (int)(col[k] >> 2), back = 4 * (tc + k * TC) - c;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (v >= back) dst[(int64_t)j * q + c + v] = acc[j][k][v];
            } else if (TC >= 64 || lane < TC) {
                const int at = TC >= 64 ? g : wave;
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(at * K + k) * 4 * TC + 4 * tc + v] = acc[j][k][v];
            }
        }
        if (groups > 1) {
            __syncthreads();
            for (int i = tid; i < 4 * nv; i += NT) {
                const int c = slot(i);
                if (i >= 4 * (nv - 1) && c < 4 * (nv - 1)) continue;
                double s = 0.0;
                for (int w = 0; w < groups; ++w) s += red[w * vs + i];
                dst[(int64_t)j * q + c] = s;
            }
            __syncthreads();
        }
    }
    // and its share of the Gram matrix; of columns that are orthonormal already, the unit matrix
    if (tid < NG) part[d.g_off + (int64_t)t.blk * kSweepGram + tid] = EXACT ? sweep_unit_gram(tid, sDrop) : sG[tid];
}

// A layer of rows shorter than a unit (q < 4): each thread takes whole rows; otherwise as above.
template <int NT, int RM>
__device__ __forceinline__ void sweep_short_body(const SweepTile &t, const SweepDesc &d, const float *Xa, const float *Xb,
                                                 const float *__restrict__ qin, double *__restrict__ part) {
    constexpr int NG = RM * (RM + 1) / 2, NS = RM * 3 + NG;
    __shared__ double sRed[NT / 64][NS], sG[NG], sR[RM][RM];
    __shared__ int sDrop[RM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = d.q, r = RM == 1 ? 1 : d.r;
    double v[RM][3], sum[NS];
#pragma unroll
    for (int j = 0; j < RM; ++j)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[j][c] = j < r && c < q ? (double)ldg1(qin + d.q_off + (int64_t)j * q + c) : 0.0;
    const bool twice = d.exact != 0;
    for (int phase = 0; phase <= (twice ? 1 : 0); ++phase) {
#pragma unroll
        for (int i = 0; i < NS; ++i) sum[i] = 0.0;
        for (int i = tid; i < t.nrows; i += NT) {
            const int row = t.row0 + i;
            double D[3], p[RM];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (c >= q) {
                    D[c] = 0.0;
                    continue;
                }
                D[c] = (double)ldg1(Xa + (int64_t)row * d.ld + c) - (double)ldg1(Xb + (int64_t)row * d.ld + c);
            }
#pragma unroll
            for (int j = 0; j < RM; ++j) p[j] = fma(D[2], v[j][2], fma(D[1], v[j][1], D[0] * v[j][0]));
            if (phase == 0) {
#pragma unroll
                for (int j = 0; j < RM; ++j)
#pragma unroll
                    for (int k = 0; k <= j; ++k) sum[RM * 3 + j * (j + 1) / 2 + k] = fma(p[k], p[j], sum[RM * 3 + j * (j + 1) / 2 + k]);
            } else {
                double ph[RM];
#pragma unroll
                for (int k = 0; k < RM; ++k) {
                    ph[k] = 0.0;
                    if (k < r) {
                        double s = p[k];
#pragma unroll
                        for (int j = 0; j < k; ++j) s -= sR[j][k] * ph[j];
                        ph[k] = sDrop[k] ? 0.0 : s / sR[k][k];
                    }
                    p[k] = (double)(float)ph[k];
                }
            }
            if (twice && phase == 0) continue;
#pragma unroll
            for (int j = 0; j < RM; ++j) {
                if (j < r) part[d.pe_off + (int64_t)j * d.p + row] = p[j];
#pragma unroll
                for (int c = 0; c < 3; ++c) sum[3 * j + c] = fma(D[c], p[j], sum[3 * j + c]);
            }
        }
        wave_sums<NS>(sum);
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < NS; ++i) sRed[wave][i] = sum[i];
        }
        __syncthreads();
        if (tid < NS) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w) s += sRed[w][tid];
            const int j = tid / 3, c = tid - 3 * j;
            if (tid < RM * 3) {
                if (phase == (twice ? 1 : 0) && j < r && c < q) part[d.qe_off + ((int64_t)t.blk * r + j) * q + c] = s;
            } else if (phase == 0) {
                sG[tid - RM * 3] = s;
            }
        }
        __syncthreads();
        if (twice && phase == 0) gram_factor<RM>(r, sG, sR, sDrop, nullptr);
    }
    if (tid < NG) part[d.g_off + (int64_t)t.blk * kSweepGram + tid] = twice ? sweep_unit_gram(tid, sDrop) : sG[tid];
}

// Vectors (q = 1) of moderate length: a wavefront does the whole power step of one (edge, layer) -- P, its norm, the unit vector rounded
// to float, the product with that -- and leaves the rounded results with a Gram sum of 1 (0: dropped), so that
// sweep_finish_kernel passes them on.
__device__ __forceinline__ void sweep_vector(const SweepDesc &d, const float *Xa, const float *Xb, const float *__restrict__ qin, double *__restrict__ part) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, p = d.p;
    const double v = (double)ldg1(qin + d.q_off);
    auto diff = [&](int row) { return (double)ldg1(Xa + (int64_t)row * d.ld) - (double)ldg1(Xb + (int64_t)row * d.ld); };
    double s = 0.0;
    for (int base = lane; base < p; base += 64 * U) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = base + 64 * u < p ? diff(base + 64 * u) * v : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) s = fma(x[u], x[u], s);
    }
    s = group_sum(s, 64);
    double floor2 = 1e-10 * s;
    if (floor2 < (double)FLT_MIN) floor2 = (double)FLT_MIN;
    const bool dropped = !(s >= floor2);
    const double norm = sqrt(s);
    double z = 0.0;
    for (int base = lane; base < p; base += 64 * U) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = base + 64 * u < p ? diff(base + 64 * u) : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + 64 * u >= p) continue;
            const float f = (float)(x[u] * v / norm);
            part[d.pe_off + base + 64 * u] = (double)f;
            z = fma(x[u], (double)f, z);
        }
    }
    z = group_sum(z, 64);
    if (lane == 0) {
        part[d.qe_off] = (double)(float)z;
        part[d.g_off] = dropped ? 0.0 : 1.0;
    }
}

// Rows too long for the registers of a work-group: P of a few rows.  Their share of D^T P is left to sweep_finish_kernel, which reads
// the rows again: as sums of a block it would be r doubles written and read per column and block, and a workspace that grows with the parameters
// (one matrix of 4096 x 70001, ring of 8, 9.2 GB: 9.2 GB of it).
template <int NT, int RM>
__device__ __forceinline__ void sweep_long_body(const SweepTile &t, const SweepDesc &d, const float *Xa, const float *Xb,
                                                const float *__restrict__ qin, double *__restrict__ part) {
    constexpr int U = 4;
    __shared__ double sRed[NT / 64][RM], sP[kSweepLongRows][RM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = d.q, r = RM == 1 ? 1 : d.r, nv = (q + 3) >> 2, last = q - 4;
    // a unit's difference; the floats before `back` belong to its neighbour
    auto diff = [&](int row, int u, double (&D)[4]) {
        float a[4], b[4];
        const uint32_t at = 4u * ((uint32_t)row * (uint32_t)d.ld + (uint32_t)min(4 * u, last));
        ld4_at(Xa, at, a);
        ld4_at(Xb, at, b);
#pragma unroll
        for (int v = 0; v < 4; ++v) D[v] = (double)a[v] - (double)b[v];
    };
    for (int m = 0; m < t.nrows; ++m) {
        double p[RM];
#pragma unroll
        for (int j = 0; j < RM; ++j) p[j] = 0.0;
        for (int u0 = tid; u0 < nv; u0 += NT * U) {
            double D[U][4];
#pragma unroll
            for (int i = 0; i < U; ++i) diff(t.row0 + m, min(u0 + i * NT, nv - 1), D[i]);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int u = u0 + i * NT, c = min(4 * u, last), back = u < nv ? 4 * u - c : 4;
#pragma unroll
                for (int j = 0; j < RM; ++j) {
                    if (j >= r) continue;
                    float w[4];
                    ld4_at(qin + d.q_off + (int64_t)j * q, 4u * (uint32_t)c, w);
#pragma unroll
                    for (int v = 0; v < 4; ++v) p[j] = fma(v < back ? 0.0 : D[i][v], (double)w[v], p[j]);
                }
            }
        }
        wave_sums<RM>(p);
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < RM; ++j) sRed[wave][j] = p[j];
        }
        __syncthreads();
        if (tid < RM) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w) s += sRed[w][tid];
            sP[m][tid] = s;
            if (tid < r) part[d.pe_off + (int64_t)tid * d.p + t.row0 + m] = s;
        }
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < RM; ++j)
#pragma unroll
            for (int i = 0; i <= j; ++i) {
                double s = 0.0;
                for (int m = 0; m < t.nrows; ++m) s = fma(sP[m][i], sP[m][j], s);
                part[d.g_off + (int64_t)t.blk * kSweepGram + j * (j + 1) / 2 + i] = s;
            }
    }
}

template <int NT, int RM>
__global__ void __launch_bounds__(NT, 2)
sweep_kernel(const SweepTile *__restrict__ tiles, int nslots, int reverse, const SweepDesc *__restrict__ descs, float *const *__restrict__ xs,
             const float *__restrict__ qstate, double *__restrict__ part) {
    extern __shared__ double smem[];
    char *lds = reinterpret_cast<char *>(smem);
    // slots of eight tiles, one per die: walked backwards slot by slot
    const int slot = (int)blockIdx.x >> 3;
    const SweepTile t = tiles[((reverse ? nslots - 1 - slot : slot) << 3) + ((int)blockIdx.x & 7)];
    if (t.nrows <= 0) return;
    if (t.blk < 0) {  // vectors: nrows consecutive (edge, layer)s from el on, a wavefront each
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        if (wave >= t.nrows) return;
        const SweepDesc d = descs[t.el + wave];
        sweep_vector(d, xs[d.wa] + d.x_off, xs[d.wb] + d.x_off, qstate, part);
        return;
    }
    const SweepDesc d = descs[t.el];
    const float *Xa = xs[d.wa] + d.x_off, *Xb = xs[d.wb] + d.x_off;
    // rows per step and steps ahead: what the registers of two work-groups of 256 per CU hold beside the sums
    if (d.q < 4) {
        sweep_short_body<NT, RM>(t, d, Xa, Xb, qstate, part);
    } else if (d.units == 0) {
        sweep_long_body<NT, RM>(t, d, Xa, Xb, qstate, part);
    } else if (d.exact) {
        if (d.units <= 1) sweep_body<NT, RM, 1, 2, 1, true>(t, d, Xa, Xb, qstate, part, lds);
        else sweep_body<NT, RM, 3, 1, 1, true>(t, d, Xa, Xb, qstate, part, lds);
    } else if (d.units <= 1) {
        sweep_body<NT, RM, 1, 4, 1, false>(t, d, Xa, Xb, qstate, part, lds);
    } else if (d.units <= 2) {
        sweep_body<NT, RM, 2, 2, 1, false>(t, d, Xa, Xb, qstate, part, lds);
    } else if (d.units <= 3) {
        sweep_body<NT, RM, 3, RM <= 2 ? 2 : 1, 1, false>(t, d, Xa, Xb, qstate, part, lds);
    } else if constexpr (RM <= 1) {
        sweep_body<NT, RM, 5, 1, 2, false>(t, d, Xa, Xb, qstate, part, lds);
    }
}

// What is left of a power step per (edge, layer): the factor R of the Gram matrix, Phat = P R^-1 and Q' = (D^T P) R^-1 by forward
// substitution, rounded to float; the column of a dropped Phat is zero and its Q column keeps its old state.  A tile is a run of
// the p rows of P followed by the q entries of Q', all r columns; the sums over the blocks run in a fixed order.  LONG (sets that have such):
// of layers whose rows are too long for the sweep's registers it forms D^T P itself, entry by entry over the rows.
template <int RM, bool LONG>
__global__ void __launch_bounds__(kThreads)
sweep_finish_kernel(const FinishTile *__restrict__ tiles, const SweepDesc *__restrict__ descs, float *const *__restrict__ xs,
                    const double *__restrict__ part, float *__restrict__ qstate, float *__restrict__ phat, int32_t *__restrict__ flags) {
    constexpr int NG = RM * (RM + 1) / 2;
    __shared__ double sG[NG];
    __shared__ double sR[RM][RM];
    __shared__ int sDrop[RM];
    const FinishTile t = tiles[blockIdx.x];
    const SweepDesc d = descs[t.el];
    const int r = RM == 1 ? 1 : d.r, tid = threadIdx.x;
    auto fetch = [&](int i, double (&v)[RM]) {  // entry i of the run, all columns
#pragma unroll
        for (int k = 0; k < RM; ++k) v[k] = 0.0;
        if (i < d.p) {
#pragma unroll
            for (int k = 0; k < RM; ++k)
                if (k < r) v[k] = part[d.pe_off + (int64_t)k * d.p + i];
        } else if (LONG && i < d.p + d.q && d.units == 0 && d.q >= 4) {
            const float *Xa = xs[d.wa] + d.x_off + (i - d.p), *Xb = xs[d.wb] + d.x_off + (i - d.p);
            constexpr int U = 8;  // rows in flight
            for (int m = 0; m < d.p; m += U) {
                float a[U], b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t at = (int64_t)min(m + u, d.p - 1) * d.ld;
                    a[u] = ldg1(Xa + at);
                    b[u] = ldg1(Xb + at);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (m + u >= d.p) continue;
#pragma unroll
                    for (int k = 0; k < RM; ++k)
                        if (k < r) v[k] = fma((double)a[u] - (double)b[u], part[d.pe_off + (int64_t)k * d.p + m + u], v[k]);
                }
            }
        } else if (i < d.p + d.q) {
            const double *src = part + d.qe_off + (i - d.p);
            const int64_t blk = (int64_t)r * d.q;
            constexpr int U = RM == 1 ? 8 : RM == 2 ? 4 : 2;  // blocks in flight
            double s[RM][U];
#pragma unroll
            for (int k = 0; k < RM; ++k)
#pragma unroll
                for (int u = 0; u < U; ++u) s[k][u] = 0.0;
            for (int b = 0; b < d.nblk; b += U) {
                double x[RM][U];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < RM; ++k) x[k][u] = b + u < d.nblk && k < r ? src[(b + u) * blk + (int64_t)k * d.q] : 0.0;
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < RM; ++k) s[k][u] += x[k][u];
            }
#pragma unroll
            for (int k = 0; k < RM; ++k) {
#pragma unroll
                for (int w = U / 2; w > 0; w >>= 1)
#pragma unroll
                    for (int u = 0; u < w; ++u) s[k][u] += s[k][u + w];
                v[k] = s[k][0];
            }
        }
    };
    double v[RM];
    int i = t.first + tid;
    fetch(i, v);
    if (tid < 64) {  // the blocks' Gram sums, a lane per block
        double gr[NG];
#pragma unroll
        for (int k = 0; k < NG; ++k) gr[k] = 0.0;
        for (int b = tid; b < d.nblk; b += 64)
#pragma unroll
            for (int k = 0; k < NG; ++k) gr[k] += part[d.g_off + (int64_t)b * kSweepGram + k];
        wave_sums<NG>(gr);
        if (tid == 0) {
#pragma unroll
            for (int k = 0; k < NG; ++k) sG[k] = gr[k];
        }
    }
    __syncthreads();
    gram_factor<RM>(r, sG, sR, sDrop, t.first == 0 ? flags + d.flag_off : nullptr);
    const int end = min(t.first + t.count, d.p + d.q);
    while (i < end) {
        double out[RM];
#pragma unroll
        for (int k = 0; k < RM; ++k) {
            out[k] = 0.0;
            if (k >= r) continue;
            double s = v[k];
#pragma unroll
            for (int j = 0; j < k; ++j) s -= sR[j][k] * out[j];
            out[k] = sDrop[k] ? 0.0 : s / sR[k][k];
            if (i < d.p) {
                phat[d.ph_off + (int64_t)k * d.p + i] = (float)out[k];
            } else {
                if (!sDrop[k]) qstate[d.q_off + (int64_t)k * d.q + i - d.p] = (float)out[k];
            }
        }
        i += kThreads;
        if (i < end) fetch(i, v);
    }
}

// ---- launches ----
template <int NT, int RM>
static void sweep_launch(const SweepLaunch &l) {
    sweep_kernel<NT, RM><<<dim3(8u * (unsigned)l.nslots), dim3(NT), (size_t)l.lds, l.stream>>>(l.tiles, l.nslots, l.reverse, l.descs, l.xs, l.qstate, l.part);
}
void launch_sweep(const SweepLaunch &l) {
    if (l.threads == 256) {
        if (l.rank <= 1) sweep_launch<256, 1>(l);
        else if (l.rank <= 2) sweep_launch<256, 2>(l);
        else sweep_launch<256, 4>(l);
    } else {
        if (l.rank <= 1) sweep_launch<512, 1>(l);
        else if (l.rank <= 2) sweep_launch<512, 2>(l);
        else sweep_launch<512, 4>(l);
    }
}
void launch_sweep_finish(const SweepLaunch &l, const FinishTile *tiles, unsigned ntiles, bool long_rows) {
#define PG_FINISH(RM) do { if (long_rows) sweep_finish_kernel<RM, true><<<dim3(ntiles), dim3(kThreads), 0, l.stream>>>(tiles, l.descs, l.xs, l.part, l.qstate, l.phat, l.flags); \
        else sweep_finish_kernel<RM, false><<<dim3(ntiles), dim3(kThreads), 0, l.stream>>>(tiles, l.descs, l.xs, l.part, l.qstate, l.phat, l.flags); } while (0)
    if (l.rank <= 1) PG_FINISH(1);
    else if (l.rank <= 2) PG_FINISH(2);
    else PG_FINISH(4);
#undef PG_FINISH
}

}  // namespace pg
