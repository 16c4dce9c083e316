// Kernels for sets of small layers.
#include "pg_device.h"
#include "pg_launch.h"

namespace pg {

// ---------------------------------------------------------------------------------------
// Small layers: everything an (edge, layer) does between two updates in one work-group.  The
// difference D = X_a - X_b is held in registers (double), so that the products, the
// orthonormalisation and any number of power steps follow each other with work-group barriers
// where the streaming kernels need a launch each.  Each worker's matrix is read once per edge.
//   Bound by the chain of loads and by instruction issue, so the code is short and free of branches per element, and all loads of a work-group
//   leave side by side (100 x 100, ring of 8: 7.8 us a launch, 10 us with a pending update; with a branch around each unit, whose load then
//   waited for the one before, 21 us).
//   Threads: TC = 2^tc_shift side by side over the units (four floats) of a row, NT / TC rows; thread (row, tc)
//   holds the units j TC + tc, j < kEdgeUnits.  A row's last unit, if it reaches past the end, is moved back to the
//   last four floats and the ones its neighbour owns are zero in D; threads past the end repeat it as zeros.
//   LDS: see edge_lds.
//   KIND kEdgeRound: `steps` power steps (Eq. (3)); kEdgeIterate: `steps` iterations of Algorithm 2, the
//   first one in R^q if `odd`.
//   PEND: X is one update behind (the last round's unit vectors phat1 and right vectors qin): every work-group
//   applies it to the values it loads, rounded as the update kernel rounds them, and for each worker one
//   of them (EdgeTile::own) stores the matrix to the other of two buffers.
// ---------------------------------------------------------------------------------------
enum EdgeKind { kEdgeRound = 0, kEdgeIterate = 1 };

// Gram-Schmidt of r columns of `len` entries (value(k, i), double) by their Gram matrix G = R^T R, with the
// dropped-column rule of gram_factor.  Every wavefront forms it for itself: no barrier.
template <int RMAX>
struct EdgeFactor {
    double R[RMAX][RMAX];  // R[k][k] = 1 for a dropped column
    bool drop[RMAX];

    template <typename F>
    __device__ __forceinline__ void form(int r, int len, F value) {
        constexpr int NG = RMAX * (RMAX + 1) / 2;
        double g[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) g[i] = 0.0;
        for (int i = threadIdx.x & 63; i < len; i += 64) {
            double v[RMAX];
#pragma unroll
            for (int k = 0; k < RMAX; ++k) v[k] = k < r ? value(k, i) : 0.0;
#pragma unroll
            for (int k = 0; k < RMAX; ++k)
#pragma unroll
                for (int j = 0; j <= k; ++j) g[k * (k + 1) / 2 + j] = fma(v[j], v[k], g[k * (k + 1) / 2 + j]);
        }
        group_sum_all<NG>(g, 64);
#pragma unroll
        for (int k = 0; k < RMAX; ++k) {
            double dk = g[k * (k + 1) / 2 + k];
#pragma unroll
            for (int j = 0; j < k; ++j) {
                double t = g[k * (k + 1) / 2 + j];
#pragma unroll
                for (int i = 0; i < j; ++i) t -= R[i][j] * R[i][k];
                R[j][k] = drop[j] ? 0.0 : t / R[j][j];
                dk -= R[j][k] * R[j][k];
            }
            double floor2 = 1e-10 * g[k * (k + 1) / 2 + k];
            if (floor2 < (double)FLT_MIN) floor2 = (double)FLT_MIN;
            drop[k] = !(dk >= floor2);
            R[k][k] = drop[k] ? 1.0 : sqrt(dk);
        }
    }
    // one row of value R^-1, rounded to float
    template <typename F>
    __device__ __forceinline__ void solve(int r, int i, F value, float (&out)[RMAX]) const {
        double ph[RMAX];
#pragma unroll
        for (int k = 0; k < RMAX; ++k) {
            double s = k < r ? value(k, i) : 0.0;
#pragma unroll
            for (int j = 0; j < k; ++j) s -= R[j][k] * ph[j];
            ph[k] = k >= r || drop[k] ? 0.0 : s / R[k][k];
            out[k] = (float)ph[k];
        }
    }
};

// NJ: units per thread; more than the layer needs repeat its last one as zeros (a branch around them would keep their
// loads from leaving side by side).
template <int NT, int RMAX, int KIND, bool PEND, int NJ>
__device__ __forceinline__ void edge_body(const EdgeTile &t, const float *Xa, const float *Xb, float *Ya, float *Yb,
                                          const ColDesc *__restrict__ cols, const float *qin, float *qout,
                                          const float *__restrict__ phat1, float *phat, int32_t *__restrict__ flags,
                                          float *pstate, float *uq, int steps, int odd, char *lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p = t.p, q = t.q, r = RMAX == 1 ? 1 : t.r;
    const int TC = 1 << t.tc_shift;
    const int tc = tid & (TC - 1), row = tid >> t.tc_shift;
    const bool rok = row < p;
    const int nv = (q + 3) >> 2, vs = 4 * nv, ps = (p + 3) & ~3;
    const int nJ = (nv + TC - 1) >> t.tc_shift;
    const EdgeLds o = edge_lds(p, q, r, t.tc_shift, NT, PEND ? t.Ra + t.Rb : 0);
    double *sRed = reinterpret_cast<double *>(lds + o.red), *sP = reinterpret_cast<double *>(lds + o.p);
    float *sV = reinterpret_cast<float *>(lds + o.v), *sPh = reinterpret_cast<float *>(lds + o.ph), *sU = reinterpret_cast<float *>(lds + o.u), *sPst = reinterpret_cast<float *>(lds + o.pst);
    const int last = max(q - 4, 0);  // where a row's last unit starts
    const uint32_t at0 = 4u * (uint32_t)(min(row, p - 1) * t.ld);
    auto col = [&](int j) { return min(4 * (j * TC + tc), last); };

    double D[NJ][4];
    {
        float x0[NJ][4], x1[NJ][4];
        if (q >= 4) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t at = at0 + 4u * (uint32_t)col(j);
                ld4_at(Xa, at, x0[j]);
                ld4_at(Xb, at, x1[j]);
            }
        } else {  // one unit per row, its missing floats repeat the last
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x0[0][v] = ld1_at(Xa, at0 + 4u * (uint32_t)min(v, q - 1));
                x1[0][v] = ld1_at(Xb, at0 + 4u * (uint32_t)min(v, q - 1));
            }
#pragma unroll
            for (int j = 1; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) x0[j][v] = x1[j][v] = 0.0f;
        }
        for (int k = 0; k < r; ++k)
            for (int c = tid; c < vs; c += NT) sV[k * vs + c] = c < q ? ldg1(qin + t.q_off + (int64_t)k * q + c) : 0.0f;
        if (KIND == kEdgeIterate) {
            for (int k = 0; k < r; ++k)
                for (int i = tid; i < p; i += NT) sPst[k * ps + i] = ldg1(pstate + t.ph_off + (int64_t)k * p + i);
        }
        if (PEND) {
            // The pending update of both workers' values, one after the other (in a loop: half the code).  Its operands are
            // staged in LDS: all loads leave side by side, and a vector is fetched once, not once per row.
            float *sQ = reinterpret_cast<float *>(lds), *sL = sQ + (t.Ra + t.Rb) * vs;
            for (int k0 = 0; k0 < t.Ra + t.Rb; k0 += 4) {
                const float *qs[4], *ls[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int j = min(k0 + k, t.Ra + t.Rb - 1);
                    const ColDesc cd = cols[j < t.Ra ? t.col_a + j : t.col_b + j - t.Ra];
                    qs[k] = qin + cd.q_off;
                    ls[k] = phat1 + cd.ph_off;
                }
                for (int i = tid; i < max(p, q); i += NT) {
                    float qv[4], lv[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        qv[k] = ldg1(qs[k] + min(i, q - 1));
                        lv[k] = ldg1(ls[k] + min(i, p - 1));
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (k0 + k < t.Ra + t.Rb && i < q) sQ[(k0 + k) * vs + i] = qv[k];
                        if (k0 + k < t.Ra + t.Rb && i < p) sL[(k0 + k) * ps + i] = lv[k];
                    }
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int side = 0; side < 2; ++side) {
                const int R = side ? t.Rb : t.Ra, col0 = side ? t.col_b : t.col_a;
                const float *sq = sQ + (side ? t.Ra * vs : 0), *sl = sL + (side ? t.Ra * ps : 0) + min(row, p - 1);
                char *Y = (char *)(side ? Yb : Ya) + at0;
                const bool store = rok && ((t.own >> side) & 1);
                constexpr int JB = 3;  // units at a time, their sums in double
#pragma unroll
                for (int jj = 0; jj < NJ; jj += JB) {
                    double xd[JB][4];
#pragma unroll
                    for (int j = 0; j < JB; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) xd[j][v] = jj + j < NJ ? (double)x0[jj + j < NJ ? jj + j : 0][v] : 0.0;
#pragma unroll 1
                    for (int k = 0; k < R; ++k) {
                        const double cp = (double)cols[col0 + k].coef * (double)sl[k * ps];
#pragma unroll
                        for (int j = 0; j < JB; ++j) {
                            if (jj + j >= NJ) continue;
                            const float4_any qv = *reinterpret_cast<const float4_any *>(sq + k * vs + col(jj + j));
#pragma unroll
                            for (int v = 0; v < 4; ++v) xd[j][v] = fma(-cp, (double)qv[v], xd[j][v]);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < JB; ++j) {
                        if (jj + j >= NJ) continue;
                        float(&x)[4] = x0[jj + j < NJ ? jj + j : 0];
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[v] = (float)xd[j][v];
                        if (store) {  // (units that overlap store the same values)
                            char *at = Y + 4u * (uint32_t)col(jj + j);
                            if (q >= 4) {
                                *(PG_GLOBAL float4_any *)at = float4_any{x[0], x[1], x[2], x[3]};
                            } else if (jj + j == 0) {
#pragma unroll
                                for (int v = 0; v < 3; ++v)
                                    if (v < q) ((PG_GLOBAL float *)at)[v] = x[v];
                            }
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float swap = x0[j][v];
                        x0[j][v] = x1[j][v];
                        x1[j][v] = swap;
                    }
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (PEND || NJ > 1) asm volatile("" : "+v"(x0[j][v]), "+v"(x1[j][v]));  // (empty: converted here, not where they are loaded)
                D[j][v] = (double)x0[j][v] - (double)x1[j][v];
            }
    }
    if (rok) {
        // floats that belong to a neighbour, or to nobody
        if (q < 4) {
#pragma unroll
            for (int v = 1; v < 4; ++v)
                if (v >= q || tc > 0) D[0][v] = 0.0;
            if (tc > 0) D[0][0] = 0.0;
        } else if ((q & 3) != 0 || NJ * TC != nv) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int back = 4 * (j * TC + tc) - col(j);
#pragma unroll
                for (int v = 0; v < 4; ++v) D[j][v] = v < back ? 0.0 : D[j][v];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) D[j][v] = 0.0;
    }
    __syncthreads();

    const int across = TC > 64 ? TC >> 6 : 1;  // wavefronts that share a row
    // P = D w for the columns w in LDS, into sP
    auto rows = [&](const float *w) {
        for (int k = 0; k < r; ++k) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float4_any w4 = *reinterpret_cast<const float4_any *>(w + k * vs + col(j));
#pragma unroll
                for (int v = 0; v < 4; ++v) s = fma(D[j][v], (double)w4[v], s);
                if (j % 3 == 2) PG_FENCE();  // registers: not all units' operands at once
            }
            s = group_sum(s, min(TC, 64));
            if ((tc & 63) == 0 && rok) {
                if (TC > 64) sRed[(k * across + (wave & (across - 1))) * ps + row] = s;
                else sP[k * ps + row] = s;
            }
        }
        __syncthreads();
        if (TC > 64) {
            for (int idx = tid; idx < r * p; idx += NT) {
                const int k = idx / p, i = idx - k * p;
                double s = 0.0;
                for (int w2 = 0; w2 < across; ++w2) s += sRed[(k * across + w2) * ps + i];
                sP[k * ps + i] = s;
            }
            __syncthreads();
        }
    };
    // sV = D^T f for column k, f this thread's entry of the unit vector: lanes that hold other rows of the same columns
    // are folded together (the four floats of a unit spread over them on the way), wavefronts meet in LDS, as many units
    // at a time as fit there.
    auto columns = [&](int k, float unit) {
        const int groups = (NT / 64) / across, group = wave / across;
        const int jb = min(edge_units_at_once(t.tc_shift, NT), nJ);
        double f = rok ? (double)unit : 0.0;
        for (int j0 = 0; j0 < nJ; j0 += jb) {
            asm volatile("" : "+v"(f));  // (empty: keeps the products of all units from being formed, and held, ahead of the loop)
            const int width = min(jb, nJ - j0) * TC * 4;
            double *dst = sRed + group * width + (TC >= 64 ? 4 * tc : TC == 32 ? 4 * tc + 2 * (lane >> 5) : 4 * tc + (lane >> 4));
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (j < j0 || j >= j0 + jb || j >= nJ) continue;
                const double a0 = D[j][0] * f, a1 = D[j][1] * f, a2 = D[j][2] * f, a3 = D[j][3] * f;
                double *at = dst + 4 * (j - j0) * TC;
                if (TC < 32) {
                    double z = fold16(fold32(a0, a2), fold32(a1, a3));
                    if (TC < 16) {
                        z += dpp_mov<0x128>(z);              // row_ror:8
                        if (TC < 8) z += dpp_mov<0x124>(z);  // row_ror:4
                        if (TC < 4) z += dpp_mov<0x4E>(z);   // quad_perm [2,3,0,1]
                        if (TC < 2) z += dpp_mov<0xB1>(z);   // quad_perm [1,0,3,2]
                    }
                    if ((lane & 15) < TC) at[0] = z;
                } else if (TC == 32) {
                    at[0] = fold32(a0, a2);
                    at[1] = fold32(a1, a3);
                } else {
                    at[0] = a0;
                    at[1] = a1;
                    at[2] = a2;
                    at[3] = a3;
                }
            }
            __syncthreads();
            // unit u's float v lies at 4 u + v; column c is float c - last of the last unit, or float c % 4 of unit c / 4
            const int first = j0 * TC * 4;
            for (int i = tid; i < width; i += NT) {
                const int c = first + i < vs - 4 ? first + i : last + (first + i - (vs - 4));
                if (c >= q || (first + i >= vs - 4 && c < vs - 4)) continue;
                double s = 0.0;
#pragma unroll 4
                for (int g = 0; g < groups; ++g) s += sRed[g * width + i];
                sV[k * vs + c] = (float)s;
            }
            __syncthreads();
        }
    };

    EdgeFactor<RMAX> fac;
    float unit[RMAX];
    bool last_odd = false;
    auto in_p = [&](int k, int i) { return sP[k * ps + i]; };
    auto in_v = [&](int k, int i) { return (double)sV[k * vs + i]; };
    auto in_pst = [&](int k, int i) { return (double)sPst[k * ps + i]; };
    for (int it = 0; it < steps; ++it, odd ^= 1) {
        if (KIND == kEdgeIterate && odd) {
            last_odd = true;
            fac.form(r, q, in_v);
            for (int c = tid; c < vs; c += NT) {
                fac.solve(r, min(c, q - 1), in_v, unit);
#pragma unroll
                for (int k = 0; k < RMAX; ++k)
                    if (k < r) sU[k * vs + c] = c < q ? unit[k] : 0.0f;
            }
            __syncthreads();
            rows(sU);
#pragma unroll
            for (int k = 0; k < RMAX; ++k)
                if (k < r && !fac.drop[k])
                    for (int i = tid; i < p; i += NT) sPst[k * ps + i] = (float)sP[k * ps + i];
            __syncthreads();
        } else {
            last_odd = false;
            if (KIND == kEdgeRound) {
                rows(sV);
                fac.form(r, p, in_p);
                fac.solve(r, min(row, p - 1), in_p, unit);
            } else {
                fac.form(r, p, in_pst);
                fac.solve(r, min(row, p - 1), in_pst, unit);
            }
            if (RMAX == 1) {
                if (!fac.drop[0]) columns(0, unit[0]);
            } else {  // one copy of the code for all columns: the entry goes through LDS, written and read by the same thread
                int keep = 0;
#pragma unroll
                for (int k = 0; k < RMAX; ++k) {
                    if (k < r) sPh[k * NT + tid] = unit[k];
                    keep |= k < r && !fac.drop[k] ? 1 << k : 0;
                }
#pragma unroll 1
                for (int k = 0; k < r; ++k)
                    if ((keep >> k) & 1) columns(k, sPh[k * NT + tid]);
            }
        }
    }
    const bool left = KIND == kEdgeRound || !last_odd;
    if (left && tc == 0 && rok) {
#pragma unroll
        for (int k = 0; k < RMAX; ++k)
            if (k < r) phat[t.ph_off + (int64_t)k * p + row] = unit[k];
    }
    for (int k = 0; k < r; ++k) {
        for (int c = tid; c < q; c += NT) {
            qout[t.q_off + (int64_t)k * q + c] = sV[k * vs + c];
            if (KIND == kEdgeIterate && last_odd) uq[t.q_off + (int64_t)k * q + c] = sU[k * vs + c];
        }
        if (KIND == kEdgeIterate) {
            for (int i = tid; i < p; i += NT) pstate[t.ph_off + (int64_t)k * p + i] = sPst[k * ps + i];
        }
    }
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < RMAX; ++k)
            if (k < r) flags[t.flag_off + k] = fac.drop[k] ? 1 : 0;
    }
}

template <int NT, int RMAX, int KIND, bool PEND, typename... Args>
__device__ __forceinline__ void edge_tile(const EdgeTile &t, Args... args) {
    const int nj = (((t.q + 3) >> 2) + (1 << t.tc_shift) - 1) >> t.tc_shift;
    if (nj <= 1) edge_body<NT, RMAX, KIND, PEND, 1>(t, args...);
    else if (nj <= 3) edge_body<NT, RMAX, KIND, PEND, 3>(t, args...);
    else if (nj <= 5) edge_body<NT, RMAX, KIND, PEND, 5>(t, args...);
    else if (nj <= 7) edge_body<NT, RMAX, KIND, PEND, 7>(t, args...);
    else edge_body<NT, RMAX, KIND, PEND, kEdgeUnits>(t, args...);
}

template <int NT, int RMAX>
__global__ void __launch_bounds__(NT)
edge_kernel(const EdgeTile *__restrict__ tiles, float *const *__restrict__ xs, const float *qin, float *qout, float *phat, int32_t *__restrict__ flags, int steps) {
    extern __shared__ double smem[];
    const EdgeTile t = tiles[blockIdx.x];
    edge_tile<NT, RMAX, kEdgeRound, false>(t, xs[t.wa] + t.x_off, xs[t.wb] + t.x_off, nullptr, nullptr, nullptr, qin, qout, nullptr,
                                           phat, flags, nullptr, nullptr, steps, 0, reinterpret_cast<char *>(smem));
}
// X one update behind: the current matrices lie in the workers' buffers (from_y = 0) or in y, `stride` floats
// per worker, and are stored, updated, to the other.
template <int NT, int RMAX>
__global__ void __launch_bounds__(NT)
edge_pending_kernel(const EdgeTile *__restrict__ tiles, const ColDesc *__restrict__ cols, float *const *__restrict__ xs,
                    float *y, int64_t stride, int from_y, const float *qin, float *qout, const float *phat1, float *phat,
                    int32_t *__restrict__ flags, int steps) {
    extern __shared__ double smem[];
    const EdgeTile t = tiles[blockIdx.x];
    float *xa = xs[t.wa] + t.x_off, *xb = xs[t.wb] + t.x_off;
    float *ya = y + t.wa * stride + t.x_off, *yb = y + t.wb * stride + t.x_off;
    edge_tile<NT, RMAX, kEdgeRound, true>(t, from_y ? ya : xa, from_y ? yb : xb, from_y ? xa : ya, from_y ? xb : yb, cols, qin, qout,
                                          phat1, phat, flags, nullptr, nullptr, steps, 0, reinterpret_cast<char *>(smem));
}
template <int NT, int RMAX>
__global__ void __launch_bounds__(NT)
edge_iterate_kernel(const EdgeTile *__restrict__ tiles, float *const *__restrict__ xs, float *q, float *pstate, float *uq,
                    float *phat, int32_t *__restrict__ flags, int iterations, int odd) {
    extern __shared__ double smem[];
    const EdgeTile t = tiles[blockIdx.x];
    edge_tile<NT, RMAX, kEdgeIterate, false>(t, xs[t.wa] + t.x_off, xs[t.wb] + t.x_off, nullptr, nullptr, nullptr, q, q, nullptr,
                                             phat, flags, pstate, uq, iterations, odd, reinterpret_cast<char *>(smem));
}

// The update that goes with them: X -= sum_j coef_j left_j right_j^T (- eta G), one unit of four floats at a
// time, in the order and with the rounding of the row kernels.  y: where X is read instead of the workers' buffers (the
// last update of a run), `stride` floats per worker; null: in place.
template <int RC, bool GRAD>
__global__ void __launch_bounds__(kThreads)
apply_kernel(const ApplyTile *__restrict__ tiles, const PairDesc *__restrict__ pairs, const ColDesc *__restrict__ cols,
             float *const *__restrict__ xs, const float *y, int64_t stride, const float *__restrict__ right,
             const float *__restrict__ left, const float *const *__restrict__ gs, double eta) {
    const ApplyTile t = tiles[blockIdx.x];
    const PairDesc pd = pairs[t.pair];
    float *X = xs[pd.worker] + pd.x_off;
    const float *S = y ? y + pd.worker * stride + pd.x_off : X;
    const float *Gp = GRAD ? gs[pd.worker] + pd.x_off : nullptr;
    const int q = pd.q, R = pd.R, nv = (q + 3) >> 2, total = pd.p * nv;
    const float *rc[RC], *lc[RC];
    double coef[RC];
#pragma unroll
    for (int j = 0; j < RC; ++j) {
        const ColDesc cd = cols[pd.col0 + min(j, R - 1)];
        rc[j] = right + cd.q_off;
        lc[j] = left + cd.ph_off;
        coef[j] = j < R ? (double)cd.coef : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kApplyUnits; ++u) {
        const int k = t.first + u * kThreads + (int)threadIdx.x;
        if (k >= total) break;
        const int row = k / nv, c = 4 * (k - row * nv);
        const int at = row * pd.ld + c, n = min(4, q - c);
        float x[4] = {0.0f, 0.0f, 0.0f, 0.0f}, g[4] = {0.0f, 0.0f, 0.0f, 0.0f}, qv[RC][4], ph[RC];
        if (n == 4) {
            ld4(S + at, x);
            if (GRAD) ld4(Gp + at, g);
#pragma unroll
            for (int j = 0; j < RC; ++j) ld4(rc[j] + c, qv[j]);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int e = min(v, n - 1);
                x[v] = ldg1(S + at + e);
                if (GRAD) g[v] = ldg1(Gp + at + e);
#pragma unroll
                for (int j = 0; j < RC; ++j) qv[j][v] = ldg1(rc[j] + c + e);
            }
        }
#pragma unroll
        for (int j = 0; j < RC; ++j) {  // (a column past the worker's counts nothing, also where the one read in its place has overflowed)
            const float l = ldg1(lc[j] + row);
            ph[j] = j < R ? l : 0.0f;
#pragma unroll
            for (int v = 0; v < 4; ++v) qv[j][v] = j < R ? qv[j][v] : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double xd = (double)x[v];
#pragma unroll
            for (int j = 0; j < RC; ++j) xd = fma(-(coef[j] * (double)ph[j]), (double)qv[j][v], xd);
            if (GRAD) xd = fma(-eta, (double)g[v], xd);
            x[v] = (float)xd;
        }
        if (n == 4) {
            *(PG_GLOBAL float4_any *)(X + at) = float4_any{x[0], x[1], x[2], x[3]};
        } else {
#pragma unroll
            for (int v = 0; v < 3; ++v)
                if (v < n) *(PG_GLOBAL float *)(X + at + v) = x[v];
        }
    }
}

// The update of sets whose workers stack different numbers of columns, in one launch: the row kernels are compiled per column count and
// access width and would follow each other, each too small to fill the chip (eight layers of odd lengths, tree of 11, rank 3: six launches).
// Bound by the fetches of
// the vectors from the caches: a thread takes the same unit of four rows, so a right vector's unit is fetched once for the four; the columns
// go by in fours, as many as the worker has.  Same operations in the same order as everywhere else.
template <bool GRAD>
__global__ void __launch_bounds__(kThreads)
apply_mixed_kernel(const MixedTile *__restrict__ tiles, const PairDesc *__restrict__ pairs, const ColDesc *__restrict__ cols,
                   float *const *__restrict__ xs, const float *y, int64_t stride, const float *__restrict__ right, const float *__restrict__ left,
                   const float *const *__restrict__ gs, double eta) {
    constexpr int M = kMixedRows;
    const MixedTile t = tiles[blockIdx.x];
    const PairDesc pd = pairs[t.pair];
    float *X = xs[pd.worker] + pd.x_off;
    const float *S = y ? y + pd.worker * stride + pd.x_off : X;
    const float *Gp = GRAD ? gs[pd.worker] + pd.x_off : nullptr;
    const int q = pd.q, R = pd.R, u1 = t.unit0 + t.nunits, end = t.row0 + t.nrows;
    const int TC = 1 << t.tc_shift, tc = threadIdx.x & (TC - 1), g = (int)threadIdx.x >> t.tc_shift, G = kThreads >> t.tc_shift;
    auto fetch = [&](const float *at, int n, float (&x)[4]) {
        if (n == 4) {
            ld4(at, x);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = ldg1(at + min(v, n - 1));
        }
    };
    for (int row = t.row0 + g * M; row < end; row += G * M)
        for (int u = t.unit0 + tc; u < u1; u += TC) {
            const int c = 4 * u, n = min(4, q - c);
            float x[M][4], gr[GRAD ? M : 1][4];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int64_t at = (int64_t)min(row + m, end - 1) * pd.ld + c;
                fetch(S + at, n, x[m]);
                if (GRAD) fetch(Gp + at, n, gr[GRAD ? m : 0]);
            }
            double xd[M][4];
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) xd[m][v] = (double)x[m][v];
            for (int k0 = 0; k0 < R; k0 += 4) {
                float qv[4][4], ph[4][M];
                double coef[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const ColDesc cd = cols[pd.col0 + min(k0 + k, R - 1)];
                    coef[k] = k0 + k < R ? (double)cd.coef : 0.0;
                    fetch(right + cd.q_off + c, n, qv[k]);
#pragma unroll
                    for (int m = 0; m < M; ++m) ph[k][m] = ldg1(left + cd.ph_off + min(row + m, end - 1));
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool on = k0 + k < R;  // (as above)
#pragma unroll
                    for (int v = 0; v < 4; ++v) qv[k][v] = on ? qv[k][v] : 0.0f;
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        const double cp = coef[k] * (double)(on ? ph[k][m] : 0.0f);
#pragma unroll
                        for (int v = 0; v < 4; ++v) xd[m][v] = fma(-cp, (double)qv[k][v], xd[m][v]);
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (row + m >= end) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (GRAD) xd[m][v] = fma(-eta, (double)gr[GRAD ? m : 0][v], xd[m][v]);
                    x[m][v] = (float)xd[m][v];
                }
                float *at = X + (int64_t)(row + m) * pd.ld + c;
                if (n == 4) {
                    *(PG_GLOBAL float4_any *)at = float4_any{x[m][0], x[m][1], x[m][2], x[m][3]};
                } else {
#pragma unroll
                    for (int v = 0; v < 3; ++v)
                        if (v < n) *(PG_GLOBAL float *)(at + v) = x[m][v];
                }
            }
        }
}

// ---- launches ----
template <int NT, int RMAX>
struct EdgeTag {
    static constexpr int nt = NT, rmax = RMAX;
};
template <int NT, typename F>
static void edge_rank(int rank, F f) {
    if (rank <= 1) f(EdgeTag<NT, 1>());
    else if (rank <= 2) f(EdgeTag<NT, 2>());
    else f(EdgeTag<NT, 4>());
}
template <typename F>
static void edge_pick(const EdgeLaunch &l, F f) {
    if (l.threads == 256) edge_rank<256>(l.rank, f);
    else edge_rank<512>(l.rank, f);
}
void launch_edge_round(const EdgeLaunch &l, const float *qin, float *qout, float *phat, int steps) {
    edge_pick(l, [&](auto tag) {
        edge_kernel<tag.nt, tag.rmax><<<dim3(l.tiles), dim3(tag.nt), (size_t)l.lds, l.stream>>>(l.d_tiles, l.d_xs, qin, qout, phat, l.d_flags, steps);
    });
}
void launch_edge_pending(const EdgeLaunch &l, const ColDesc *cols, float *y, int64_t stride, bool from_y, const float *qin, float *qout,
                         const float *before, float *phat, int steps) {
    edge_pick(l, [&](auto tag) {
        edge_pending_kernel<tag.nt, tag.rmax><<<dim3(l.tiles), dim3(tag.nt), (size_t)l.lds, l.stream>>>(
            l.d_tiles, cols, l.d_xs, y, stride, from_y ? 1 : 0, qin, qout, before, phat, l.d_flags, steps);
    });
}
void launch_edge_iterate(const EdgeLaunch &l, float *q, float *pstate, float *uq, float *phat, int iterations, bool odd) {
    edge_pick(l, [&](auto tag) {
        edge_iterate_kernel<tag.nt, tag.rmax><<<dim3(l.tiles), dim3(tag.nt), (size_t)l.lds, l.stream>>>(
            l.d_tiles, l.d_xs, q, pstate, uq, phat, l.d_flags, iterations, odd ? 1 : 0);
    });
}
void launch_apply(int cols_compiled, unsigned ntiles, hipStream_t stream, const ApplyTile *tiles, const PairDesc *pairs, const ColDesc *cols,
                  float *const *xs, const float *y, int64_t stride, const float *right, const float *left, const float *const *gs, double eta) {
#define PG_APPLY(RC) do { if (gs) apply_kernel<RC, true><<<dim3(ntiles), dim3(kThreads), 0, stream>>>(tiles, pairs, cols, xs, y, stride, right, left, gs, eta); \
        else apply_kernel<RC, false><<<dim3(ntiles), dim3(kThreads), 0, stream>>>(tiles, pairs, cols, xs, y, stride, right, left, gs, eta); } while (0)
    if (cols_compiled <= 1) PG_APPLY(1);
    else if (cols_compiled <= 2) PG_APPLY(2);
    else if (cols_compiled <= 4) PG_APPLY(4);
    else PG_APPLY(8);  // (more: launch_apply_mixed)
#undef PG_APPLY
}

void launch_apply_mixed(unsigned ntiles, hipStream_t stream, const MixedTile *tiles, const PairDesc *pairs, const ColDesc *cols,
                        float *const *xs, const float *y, int64_t stride, const float *right, const float *left, const float *const *gs, double eta) {
    if (gs) apply_mixed_kernel<true><<<dim3(ntiles), dim3(kThreads), 0, stream>>>(tiles, pairs, cols, xs, y, stride, right, left, gs, eta);
    else apply_mixed_kernel<false><<<dim3(ntiles), dim3(kThreads), 0, stream>>>(tiles, pairs, cols, xs, y, stride, right, left, gs, eta);
}

}  // namespace pg
