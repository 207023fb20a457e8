// Tall-skinny FP64 products over the grid on the matrix cores: the overlap
// Gram matrix G = dV psi psi^T and the adjoint contraction B = Gam psi^T
// (N x M times M x N, reductions over the M grid nodes), and the orbital
// transform phi = Q psi (N x N times N x M).  Eq. 6-8 and Sec. I.B give the
// products; N <= 128 orbitals of one spin channel, M up to 2^29 nodes.  All
// channels of a batch whose N takes the same number of 16-row tiles share a
// launch.
//
// All three are bound by the reads (and, for phi, writes) of the fields:
// there is no staging, a wave takes its operands from memory in the layout
// the matrix cores want and keeps every sum it can in registers.  In the
// reductions lane (row c = l % 16, g = l / 16) holds nodes 4 g .. 4 g + 3 of
// its row (32 contiguous bytes; the four lanes of a row read a 128-byte
// line), and k step j contracts node 4 g + j: any assignment of nodes to
// k steps splits the sum, as long as both operands use it.
#include <algorithm>
#include <array>
#include <map>
#include <mutex>

#include "kernels.h"
#include "lds.h"

namespace fsic {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
// 16 bytes at any 8-byte boundary (rows of an odd number of nodes)
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// channel of a block: prod.c[i].b0 are ascending
__device__ __forceinline__ int channel_of(const ProdBatch &p, int b) {
    int c = 0;
    while (c + 1 < p.n && b >= p.c[c + 1].b0) ++c;
    return c;
}

}  // namespace

// part[block] = sum over the block's 16-node groups of X_i(m) Y_j(m), as
// 16 x 16 tiles.  T: row tiles of a wave; GW = 1: N <= 16 T, every wave forms
// all tiles over its own groups and the four sums are added in LDS; GW = 2:
// N <= 32 T, wave (w / 2, w % 2) forms its quarter over all the block's
// groups.  SYM: Y = X, only tile pairs t1 <= t2.  Above 96 orbitals (T = 4) the
// 16 accumulator tiles spill 92 B a lane (SYM) and 32 B.
template <int T, int GW, bool SYM>
__global__ __launch_bounds__(256, 2) void k_nt(ProdBatch prod, double *part) {
    const int ci = channel_of(prod, blockIdx.x);
    const ProdChan ch = prod.c[ci];
    const int N = ch.N;
    const long long M = ch.M;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int wi = GW == 2 ? w >> 1 : 0, wj = GW == 2 ? w & 1 : 0;
    constexpr int NT = T * GW, NP = 16 * NT;  // tiles and rows of a partial tile
    const bool same = SYM && wi == wj;        // X and Y rows are the same
    const int b = blockIdx.x - ch.b0;
    const long long groups = (M + 15) >> 4;
    const long long g0 = groups * b / ch.nblk, g1 = groups * (b + 1) / ch.nblk;
    dbl4 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = dbl4{0.0, 0.0, 0.0, 0.0};
    const double *const Y = SYM ? ch.X : ch.Y;
    const int step = GW == 2 ? 1 : 4;
    const bool idle = SYM && GW == 2 && wi > wj;
    auto products = [&](const double (&x)[T][4], const double (&y)[T][4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int t = 0; t < T; ++t)
                    if (!(SYM && GW == 1 && t < a)) acc[a][t] = mfma(x[a][j], y[t][j], acc[a][t]);
    };
    // Whole groups: PD of them in flight, in loads that no branch holds (one in
    // a branch is waited for where the branches meet).  Rows past N read row
    // N - 1; their sums are not used.  With this and four groups a wave
    // instead of sixteen, 5 orbitals on 40^3: B 20.4 -> 5.0 us, G 11.3 -> 4.4;
    // 45 on 80^3: G 47 -> 34; large fields are at their bytes either way (four
    // groups in flight instead of two: 96^3 G 41 -> 46 us).
    constexpr int PD = T <= 2 ? 2 : 1;
    const double *px[T], *py[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        px[t] = ch.X + (long long)min(16 * (T * wi + t) + c, N - 1) * M + 4 * g;
        py[t] = Y + (long long)min(16 * (T * wj + t) + c, N - 1) * M + 4 * g;
    }
    auto load = [&](const double *const (&p)[T], long long grp, double (&f)[T][4]) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const dbl2u lo = *reinterpret_cast<const dbl2u *>(p[t] + 16 * grp);
            const dbl2u hi = *reinterpret_cast<const dbl2u *>(p[t] + 16 * grp + 2);
            f[t][0] = lo.x;
            f[t][1] = lo.y;
            f[t][2] = hi.x;
            f[t][3] = hi.y;
        }
    };
    const long long g1f = std::min(g1, M >> 4);
    const long long first = g0 + (GW == 2 ? 0 : w);
    if (first < g1f && !idle) {
        const long long last = g1f - 1;
        double x[PD][T][4], y[PD][T][4];
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            load(px, std::min(first + u * step, last), x[u]);
            if (!same) load(py, std::min(first + u * step, last), y[u]);
        }
        for (long long q = first; q < g1f; q += PD * step) {
#pragma unroll
            for (int u = 0; u < PD; ++u) {
                double xc[T][4], yc[T][4];
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        xc[t][j] = x[u][t][j];
                        yc[t][j] = same ? x[u][t][j] : y[u][t][j];
                    }
                const long long nq = std::min(q + (PD + u) * step, last);
                load(px, nq, x[u]);
                if (!same) load(py, nq, y[u]);
                if (q + u * step < g1f) products(xc, yc);
            }
        }
    }
    // the nodes after the last whole group
    if (g1 > g1f && (GW == 2 ? !idle : (int)((g1f - g0) & 3) == w)) {
        double x[T][4], y[T][4];
        const long long m = 16 * g1f + 4 * g;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[t][j] = m + j < M ? px[t][16 * g1f + j] : 0.0;
                y[t][j] = m + j < M ? py[t][16 * g1f + j] : 0.0;
            }
        products(x, y);
    }
    double *out = part + ch.poff + (size_t)b * NP * NP;
    if (GW == 2) {
        if (!idle)
#pragma unroll
            for (int a = 0; a < T; ++a)
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        out[(size_t)(16 * (T * wi + a) + g + 4 * j) * NP + 16 * (T * wj + t) + c] = acc[a][t][j];
        return;
    }
    __shared__ double sx[4][256];
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (SYM && t < a) continue;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 4; ++j) sx[w][64 * j + lane] = acc[a][t][j];
            __syncthreads();
            // wave w writes accumulator element w
            const int e = 64 * w + lane;
            out[(size_t)(16 * a + g + 4 * w) * NP + 16 * t + c] = (sx[0][e] + sx[1][e]) + (sx[2][e] + sx[3][e]);
        }
}

// out[i][j] = scale sum of a channel's partial tiles (SYM: from the upper
// tile triangle), added in a fixed order; 32 elements of a row and 32 runs of
// partials per block
template <bool SYM>
__global__ __launch_bounds__(1024) void k_nt_final(ProdBatch prod, int NP, const double *part) {
    __shared__ double sx[32][33];
    const ProdChan ch = prod.c[blockIdx.z];
    const int N = ch.N, i = blockIdx.y, j = 32 * blockIdx.x + (threadIdx.x & 31), run = threadIdx.x >> 5;
    if (i >= N || 32 * (int)blockIdx.x >= N) return;  // uniform
    // SYM: entries below the diagonal's tiles are written with their mirror
    // image (reading them here, down a column of every partial tile: 2 x 32
    // orbitals 35 -> 9 us, 45 orbitals 21 -> 5 us)
    const bool own = j < N && !(SYM && (i >> 4) > (j >> 4));
    double s = 0.0;
    if (own) {
        const double *p = part + ch.poff + (size_t)i * NP + j;
#pragma unroll 4
        for (int b = run; b < ch.nblk; b += 32) s += p[(size_t)b * NP * NP];
    }
    sx[run][threadIdx.x & 31] = s;
    __syncthreads();
    if (run == 0 && own) {
        s = 0.0;
        for (int r = 0; r < 32; ++r) s += sx[r][threadIdx.x];
        ch.out[(size_t)i * N + j] = ch.scale * s;
        if (SYM && (i >> 4) < (j >> 4)) ch.out[(size_t)j * N + i] = ch.scale * s;
    }
}

// out[i][m] = sum_a A[i][a] X_a(m).  A wave takes 32 nodes: lane c holds nodes
// 2 c and 2 c + 1 of its k rows, so loads and stores are 16 bytes a lane and
// 256 bytes a row.  The fragments of A stay in registers (T <= 2) or LDS.
// (One 16-node strip at a time with A read through the cache took 526 us for
// 32 orbitals at 128^3; the fields' bytes take 210.)  12 to 28 B a lane are
// spilled at T = 3, 7 and 8.
template <int T>
__global__ __launch_bounds__(256, 2) void k_nn(ProdBatch prod) {
    extern __shared__ __attribute__((aligned(16))) double af_lds[];
    const ProdChan ch = prod.c[channel_of(prod, blockIdx.x)];
    const int N = ch.N;
    const long long M = ch.M;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    constexpr bool REG = T <= 2;
    const int ks = (N + 3) >> 2;
    double af[REG ? T : 1][REG ? 4 * T : 1];
    auto A = [&](int t, int s) {
        const int i = 16 * t + c, a = 4 * s + g;
        return i < N && a < N ? ch.A[(size_t)i * N + a] : 0.0;
    };
    if constexpr (REG) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) af[t][s] = A(t, s);
    } else {
        for (int e = w; e < T * 4 * T; e += 4) af_lds[64 * e + lane] = A(e / (4 * T), e % (4 * T));
        __syncthreads();
    }
    const long long strips = (M + 31) >> 5;
    const long long wave = 4LL * (blockIdx.x - ch.b0) + w, nwave = 4LL * ch.nblk;
    // k rows in chunks of CH steps: the next one (of this strip or the wave's
    // next) is loaded while this one is used
    constexpr int CH = T <= 3 ? 4 * T : T == 4 ? 8 : 4, NCH = 4 * T / CH;
    double bn[CH][2];
    auto load = [&](long long st, int q) {
        const long long m = 32 * st + 2 * c;
        const bool in2 = m + 2 <= M, in1 = m < M;
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int a = 4 * (CH * q + s) + g;
            const double *p = ch.X + (long long)a * M + m;
            if (a < N && in2) {
                const dbl2u v = *reinterpret_cast<const dbl2u *>(p);
                bn[s][0] = v.x;
                bn[s][1] = v.y;
            } else {
                bn[s][0] = a < N && in1 ? p[0] : 0.0;
                bn[s][1] = 0.0;
            }
        }
    };
    if (wave < strips) load(wave, 0);
    for (long long st = wave; st < strips; st += nwave) {
        const long long m = 32 * st + 2 * c;
        const bool in2 = m + 2 <= M, in1 = m < M;
        dbl4 acc[T][2];
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t][0] = acc[t][1] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
        for (int q = 0; q < NCH; ++q) {
            double b[CH][2];
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                b[s][0] = bn[s][0];
                b[s][1] = bn[s][1];
            }
            if (q + 1 < NCH) load(st, q + 1);
            else if (st + nwave < strips) load(st + nwave, 0);
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                if (REG && s >= 4 * (T - 1) && s >= ks) continue;  // uniform
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    double a;
                    if constexpr (REG) a = af[t][s];
                    else a = af_lds[64 * (t * 4 * T + CH * q + s) + lane];
                    acc[t][0] = mfma(a, b[s][0], acc[t][0]);
                    acc[t][1] = mfma(a, b[s][1], acc[t][1]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * t + g + 4 * r;
                double *p = ch.out + (long long)i * M + m;
                if (i < N && in2) {
                    dbl2u v;
                    v.x = acc[t][0][r];
                    v.y = acc[t][1][r];
                    *reinterpret_cast<dbl2u *>(p) = v;
                } else if (i < N && in1) {
                    p[0] = acc[t][0][r];
                }
            }
    }
}

namespace {

int cu_count() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) return 256;
    return v;
}

int tiles_of(int N) { return (N + 15) / 16; }
// (T, GW) of a reduction over N rows
void nt_shape(int N, int &T, int &GW) {
    const int t = tiles_of(N);
    GW = t <= 3 ? 1 : 2;
    T = GW == 1 ? t : (t + 1) / 2;
}

// Blocks of a channel's reduction: what the device holds at once (more would
// only add partial tiles), at least four 16-node groups for each wave.  They
// depend on the channel, the device and the room for partial tiles (fit), not
// on the batch: S of nearly dependent orbitals carries the order of these sums
// into the forces, and a system gives the same S alone and in a batch.  A
// context has room for all blocks it could use at any N; above 64 orbitals
// fsic_op_flo and fsic_op_flo_noalloc have less, so the last bits of their G
// may differ from a context's.
long long nt_blocks(int T, int GW, long long M, size_t fit) {
    const long long occ = GW == 1 && T <= 2 ? 4 : 2;
    // four groups a wave at least: fields of few nodes are bound by latency
    const long long most = std::max<long long>(1, M / (GW == 1 ? 256 : 64));
    return std::max<long long>(1, std::min({most, occ * cu_count(), (long long)fit}));
}

template <bool SYM>
hipError_t nt_run(ProdBatch &p, int T, int GW, int nmax, double *part, hipStream_t s) {
    const size_t NP = 16 * (size_t)T * GW;
    const int blocks = p.c[p.n - 1].b0 + p.c[p.n - 1].nblk;
#define GO(TT, GG) hipLaunchKernelGGL((k_nt<TT, GG, SYM>), dim3(blocks), dim3(256), 0, s, p, part)
    if (GW == 1) {
        if (T == 1) GO(1, 1);
        else if (T == 2) GO(2, 1);
        else GO(3, 1);
    } else {
        if (T == 2) GO(2, 2);
        else if (T == 3) GO(3, 2);
        else GO(4, 2);
    }
#undef GO
    hipLaunchKernelGGL((k_nt_final<SYM>), dim3((nmax + 31) / 32, nmax, p.n), dim3(1024), 0, s, p, (int)NP, part);
    p = ProdBatch{};
    return hipGetLastError();
}

// the channels of each shape in as few launches as their partial tiles and
// the argument block allow
template <bool SYM>
hipError_t nt_launch(const ProdChan *chans, int n, double *part, size_t cap, hipStream_t s) {
    for (int T = 1; T <= 4; ++T)
        for (int GW = 1; GW <= 2; ++GW) {
            const size_t NP = 16 * (size_t)T * GW, fit = cap / (NP * NP);
            if (fit < 1) continue;
            ProdBatch p{};
            int nmax = 0;
            size_t used = 0;
            for (int i = 0; i < n; ++i) {
                int t, gw;
                nt_shape(chans[i].N, t, gw);
                if (t != T || gw != GW) continue;
                const int nblk = (int)nt_blocks(T, GW, chans[i].M, fit);
                if (p.n == kProdBatch || (p.n && used + nblk > fit)) {
                    const hipError_t e = nt_run<SYM>(p, T, GW, nmax, part, s);
                    if (e != hipSuccess) return e;
                    nmax = 0;
                    used = 0;
                }
                ProdChan &c = p.c[p.n];
                c = chans[i];
                c.nblk = nblk;
                c.b0 = (int)used;
                c.poff = used * NP * NP;
                used += nblk;
                nmax = std::max(nmax, c.N);
                ++p.n;
            }
            if (p.n) {
                const hipError_t e = nt_run<SYM>(p, T, GW, nmax, part, s);
                if (e != hipSuccess) return e;
            }
        }
    return hipSuccess;
}

bool bad(const ProdChan *chans, int n) {
    for (int i = 0; i < n; ++i)
        if (chans[i].N < 1 || chans[i].N > kMaxOrb || chans[i].M < 1) return true;
    return false;
}

}  // namespace

hipError_t launch_gram(const ProdChan *chans, int n, double *part, size_t cap, hipStream_t s) {
    if (bad(chans, n)) return hipErrorInvalidValue;
    return nt_launch<true>(chans, n, part, cap, s);
}

hipError_t launch_contract(const ProdChan *chans, int n, double *part, size_t cap, hipStream_t s) {
    if (bad(chans, n)) return hipErrorInvalidValue;
    return nt_launch<false>(chans, n, part, cap, s);
}

hipError_t launch_transform(const ProdChan *chans, int n, hipStream_t s) {
    if (bad(chans, n)) return hipErrorInvalidValue;
    for (int T = 1; T <= 8; ++T)
        for (int i0 = 0; i0 < n;) {
            ProdBatch p{};
            for (; i0 < n && p.n < kProdBatch; ++i0)
                if (tiles_of(chans[i0].N) == T) p.c[p.n++] = chans[i0];
            if (!p.n) continue;
            const size_t lds = T <= 2 ? 0 : (size_t)T * 4 * T * 64 * sizeof(double);
            // what the compute units hold at once, shared by work (each
            // node's sums are its own: the split does not matter)
            const double occ = T <= 2 ? 4.0 : T <= 6 ? 2.0 : 1.0;
            double work = 0.0;
            for (int i = 0; i < p.n; ++i) work += (double)p.c[i].M * p.c[i].N;
            int blocks = 0;
            for (int i = 0; i < p.n; ++i) {
                const double share = occ * cu_count() * ((double)p.c[i].M * p.c[i].N) / work;
                p.c[i].nblk = (int)std::max(1.0, std::min(std::ceil(p.c[i].M / 128.0), std::floor(share + 0.5)));
                p.c[i].b0 = blocks;
                blocks += p.c[i].nblk;
            }
#define GO(TT)                                                                                                  \
    case TT:                                                                                                    \
        if (const hipError_t e = allow_lds((const void *)k_nn<TT>, lds)) return e;                              \
        hipLaunchKernelGGL((k_nn<TT>), dim3(blocks), dim3(256), lds, s, p);                                     \
        break;
            switch (T) { GO(1) GO(2) GO(3) GO(4) GO(5) GO(6) GO(7) GO(8) }
#undef GO
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

}  // namespace fsic
