// Transition statistics (eq 41) and the look-ahead cost-to-go Phi (eq 42) on
// the device, for every layer of a stack.  The results equal the host
// library's ordermoe_estimate_transitions and ordermoe_build_lookahead bit for
// bit: counts are integers (atomic increments commute), each probability is
// one fp64 division of a count by its row total, every candidate cost is
// formed with the same fp64 operations in the same order (no contraction), a
// minimum of doubles does not depend on the order it is taken in, and each
// Phi entry is a dot product summed in target order.
//
//   transition_rows_kernel     short calibrations: counts of a few rows of one
//                              layer pair in LDS, then P = n / total
//   fill_u32, transition_count_kernel, transition_norm_kernel
//                              long calibrations: counts in device memory
//   lookahead_depth_kernel     one depth h, one block per (layer l, source s):
//                              V[r'] = min over the next layer's candidates of
//                              target r' from source s of g_{l+1}(m', k' | s) +
//                              Phi^(h-1)_{l+1}(m', k'), then Phi^(h)_l[s][k] =
//                              sum_r' P_l[k][r'] V[r']
//   fill_f64                   zeros where there is no depth to run (a kernel,
//                              not a memset, so that the call can be captured)
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"

namespace ordermoe {
namespace {

constexpr int LA_THREADS = 256;
constexpr int LA_WAVES = LA_THREADS / 64;

__global__ void __launch_bounds__(LA_THREADS) fill_f64(double* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * LA_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * LA_THREADS)
        p[i] = 0.0;
}

__global__ void __launch_bounds__(LA_THREADS) fill_u32(uint32_t* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * LA_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * LA_THREADS)
        p[i] = 0u;
}

// ids outside [0, E) are not counted
__global__ void __launch_bounds__(LA_THREADS) transition_count_kernel(const int32_t* top1, int32_t N, int32_t E,
                                                                      int64_t T_cal, uint32_t* cnt) {
    const int64_t n = (int64_t)(N - 1) * T_cal;
    for (int64_t i = (int64_t)blockIdx.x * LA_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * LA_THREADS) {
        const int64_t l = i / T_cal, t = i - l * T_cal;
        const int32_t a = top1[l * T_cal + t], b = top1[(l + 1) * T_cal + t];
        if (a >= 0 && a < E && b >= 0 && b < E) atomicAdd(&cnt[(l * E + a) * E + b], 1u);
    }
}

// one wave per row: the row total by a shuffle sum, then the quotients
__global__ void __launch_bounds__(LA_THREADS) transition_norm_kernel(const uint32_t* cnt, int32_t N, int32_t E,
                                                                     double* P) {
    const int lane = threadIdx.x & 63;
    const int64_t rows = (int64_t)(N - 1) * E;
    for (int64_t row = (int64_t)blockIdx.x * LA_WAVES + (threadIdx.x >> 6); row < rows;
         row += (int64_t)gridDim.x * LA_WAVES) {
        const uint32_t* c = cnt + row * E;
        int64_t tot = 0;
        for (int k = lane; k < E; k += 64) tot += c[k];
        for (int off = 32; off >= 1; off >>= 1) tot += __shfl_xor(tot, off);
        for (int k = lane; k < E; k += 64) P[row * E + k] = tot > 0 ? (double)c[k] / (double)tot : 0.0;
    }
}

// Rows [r0, r0 + R) of layer pair l, counted in LDS: the block reads all of the
// pair's tokens and keeps those whose first expert falls in its rows, so one
// launch replaces the clear, the atomics in device memory and the division
// pass, whose serial row sums per thread took 56 of the 64 us (32 layers of
// 128 experts, 2048 tokens); 5.5 us now.
constexpr int TR_LDS_COUNTS = 8192;         // counts of one block, 32 KB
constexpr int64_t TR_MAX_T = 32768;         // the longest calibration counted this way

__global__ void __launch_bounds__(LA_THREADS) transition_rows_kernel(const int32_t* top1, int32_t E, int32_t R,
                                                                     int32_t nb, int64_t T_cal, double* P) {
    __shared__ uint32_t s_cnt[TR_LDS_COUNTS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l = (int)(blockIdx.x / nb), r0 = (int)(blockIdx.x % nb) * R;      // nb blocks per layer pair
    const int nr = E - r0 < R ? E - r0 : R;
    for (int i = tid; i < nr * E; i += LA_THREADS) s_cnt[i] = 0u;
    __syncthreads();
    const int32_t* ta = top1 + (int64_t)l * T_cal;
    const int32_t* tb = ta + T_cal;
    constexpr int U = 8;                    // tokens in flight per thread
    for (int64_t t0 = tid; t0 < T_cal; t0 += U * LA_THREADS) {
        int32_t a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = t0 + u * LA_THREADS;
            a[u] = t < T_cal ? ta[t] : -1;
            b[u] = t < T_cal ? tb[t] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (a[u] >= r0 && a[u] < r0 + nr && b[u] >= 0 && b[u] < E) atomicAdd(&s_cnt[(a[u] - r0) * E + b[u]], 1u);
    }
    __syncthreads();
    for (int r = wave; r < nr; r += LA_WAVES) {
        int64_t tot = 0;
        for (int k = lane; k < E; k += 64) tot += s_cnt[r * E + k];
        for (int off = 32; off >= 1; off >>= 1) tot += __shfl_xor(tot, off);
        double* p = P + ((int64_t)l * E + r0 + r) * E;
        for (int k = lane; k < E; k += 64) p[k] = tot > 0 ? (double)s_cnt[r * E + k] / (double)tot : 0.0;
    }
}

struct LookArgs {
    int32_t N, E, M;
    const double* P;          // [N-1][E][E]
    const uint8_t* x;         // [N][M][E]
    const float* sim;         // [N][E][E]
    const int32_t* group_of;  // [N][E]
    const float* theta;       // [N]
    const double* z_bits;     // [N]
    const double* c;          // [N][E]
    const double* d_ref;      // [N]
    const double* B;          // [M][M]
    const double* tau;        // [M][M]
    const double* F;          // [M]
    double omega_T, omega_Q;
    float Qbar;
    int32_t pin, allow_sub;
};

// eq 37's per-step delay of (m, k) from source s
__device__ inline double step_delay_dev(const LookArgs& a, int s, int m, int k, double z, const double* cl) {
    const double trans = (s != m) ? (z / a.B[(size_t)s * a.M + m] + a.tau[(size_t)s * a.M + m]) : 0.0;
    return trans + cl[k] / a.F[m];
}

// Phi^(h) of one (layer l, source s) per block; layer N-1 is zero.  What bounds
// it is latency, so everything shared is formed once and read from LDS: the
// delay part of the cost of every (m', k') at layer l + 1 (three fp64 divisions
// each), the servers of each k' as a mask, and the members of each target's
// group as a bit mask, so that a thread (one target r') visits its few
// candidates instead of scanning all E x M pairs with the divisions inside the
// scan.  The candidates are visited in (k', m') order with the same fp64
// operations per candidate, and the products of a Phi entry are added in r'
// order, so the values do not depend on this layout.  P_l is staged in LDS
// LA_PC columns at a time, which makes its reads whole lines.  One depth of 32
// layers of 128 experts on 8 servers: 248 us for the minima and 21 us for the
// sums before, 15 us for both now (about 3 us group masks, 2 us costs, 3 us
// minima, 5 us sums).
constexpr int LA_PC = 64, LA_LP = LA_PC + 2;   // columns per step, doubles per staged row (16-byte rows)
typedef double f64x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t LA_OOR = 0x80000000u;    // offset past every buffer: reads zero
constexpr int LD_THREADS = 512, LD_WAVES = LD_THREADS / 64;

__host__ __device__ inline size_t lookahead_lds_cost(int E, int M) {
    const size_t cost = (size_t)2 * M * E, tile = (size_t)E * LA_LP;   // doubles; the tile replaces the costs
    return ((cost > tile ? cost : tile) + 1) & ~size_t(1);
}
size_t lookahead_lds(int E, int M) {
    return (lookahead_lds_cost(E, M) + E + (size_t)E * ((E + 63) / 64)) * sizeof(double) + (size_t)E * sizeof(uint32_t);
}

__global__ void __launch_bounds__(LD_THREADS) lookahead_depth_kernel(const LookArgs a, const double* prev,
                                                                     double* cur) {
    extern __shared__ __attribute__((aligned(16))) double s_la[];
    const int E = a.E, M = a.M;
    const int64_t ME = (int64_t)M * E;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks go to the 8 XCDs in turn: the M blocks of a layer, which read the
    // same P and similarities, sit on one of them and share its L2
    const int j8 = (int)blockIdx.x >> 3;
    const int l = (j8 / M) * 8 + ((int)blockIdx.x & 7), s = j8 % M;
    if (l >= a.N) return;
    double* out = cur + (int64_t)l * ME + (int64_t)s * E;
    if (l == a.N - 1) {
        for (int k = tid; k < E; k += LD_THREADS) out[k] = 0.0;
        return;
    }
    double* s_v0 = s_la;                                   // [M][E] delay part of the cost
    double* s_nxt = s_la + ME;                             // [M][E] Phi^(h-1) of layer l + 1
    double* s_P = s_la;                                    // [E][LA_LP], after the minima
    double* s_V = s_la + lookahead_lds_cost(E, M);         // [E]
    const int NW = (E + 63) >> 6;                          // 64-expert words of a member mask
    uint64_t* s_mem = (uint64_t*)(s_V + E);                // [E][NW] members of each expert's group
    uint32_t* s_mask = (uint32_t*)(s_mem + E * NW);        // [E] servers of each expert
    const int l1 = l + 1;
    const uint8_t* xl = a.x + (size_t)l1 * ME;
    const float* sl = a.sim + (size_t)l1 * E * E;
    const double* cl = a.c + (size_t)l1 * E;
    const double z = a.z_bits[l1], dref = a.d_ref[l1];
    for (int k = tid; k < E; k += LD_THREADS) s_mask[k] = 0;
    const bool subs = a.allow_sub && a.Qbar > 0.0f;
    const float th = a.theta[l1];
    {
        // group masks by ballots: every wave holds all group ids, 64 per register
        constexpr int W = ORDERMOE_MAX_EXPERTS / 64;
        int32_t g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int k = w * 64 + lane;
            g[w] = a.group_of[(size_t)l1 * E + (k < E ? k : E - 1)];
        }
#pragma unroll
        for (int wr = 0; wr < W; ++wr)
            for (int i = wave; i < 64 && wr * 64 + i < E; i += LD_WAVES) {
                const int r = wr * 64 + i;
                const int32_t gr = __builtin_amdgcn_readlane(g[wr], i);
#pragma unroll
                for (int w = 0; w < W; ++w)
                    if (w < NW) {
                        const uint64_t b = subs ? __ballot(g[w] == gr && w * 64 + lane < E) : w == wr ? 1ull << i : 0ull;
                        if (lane == 0) s_mem[r * NW + w] = b;
                    }
            }
    }
    __syncthreads();
    // thread r1's candidate experts (the target and its group mates) in
    // increasing order; the similarities of the first four are read here
    struct Members {
        uint64_t mem;
        int w;
    } it{0, -1};
    const int r1 = tid;
    auto next = [&]() -> int {                                 // -1: no more
        while (!it.mem && it.w + 1 < NW) it.mem = s_mem[r1 * NW + ++it.w];
        if (!it.mem) return -1;
        const int k1 = it.w * 64 + __builtin_ctzll(it.mem);
        it.mem &= it.mem - 1;
        return k1;
    };
    int kk[4];
    float sv[4];
    auto four = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) kk[u] = next();
#pragma unroll
        for (int u = 0; u < 4; ++u) sv[u] = sl[(size_t)r1 * E + (kk[u] >= 0 ? kk[u] : 0)];
    };
    if (r1 < E) four();
    // four (m', k') per thread and pass, their reads issued together (reads
    // past the table re-read its last entry and are discarded)
    for (int i0 = tid; i0 < (int)ME; i0 += 4 * LD_THREADS) {
        uint8_t xv[4];
        double nx[4], dl[4];
        int im[4], ik[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * LD_THREADS < (int)ME ? i0 + u * LD_THREADS : (int)ME - 1;
            im[u] = i / E;
            ik[u] = i - im[u] * E;
            xv[u] = xl[i];
            nx[u] = prev ? prev[(size_t)l1 * ME + i] : 0.0;
            dl[u] = step_delay_dev(a, s, im[u], ik[u], z, cl);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * LD_THREADS;
            if (i < (int)ME) {
                s_v0[i] = a.omega_T * dl[u] / dref;                                     // eq 38
                s_nxt[i] = nx[u];
                if (xv[u]) atomicOr(&s_mask[ik[u]], 1u << im[u]);
            }
        }
    }
    __syncthreads();
    // LA_PC columns of P_l per step, a row per wave and read, the reads of the
    // next step in flight while this one is summed (and the first ones during
    // the minima); rows and columns past E read zeros and are never stored
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(a.P + (size_t)l * E * E), (short)0, E * E * (int)sizeof(double), 0x00020000);
    constexpr int PH = ORDERMOE_MAX_EXPERTS / LD_WAVES / 2;
    double pv[2 * PH];
    auto pread = [&](int c0) {
        const uint32_t col = c0 + lane < E ? (uint32_t)(c0 + lane) * 8u : LA_OOR;
        const uint32_t rstep = (uint32_t)(LD_WAVES * E) * 8u, r0 = (uint32_t)(wave * E) * 8u;
        auto rd = [&](int u) {
            return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rp, (int)(col + r0 + (uint32_t)u * rstep), 0, 0));
        };
#pragma unroll
        for (int u = 0; u < PH; ++u) pv[u] = rd(u);
        if (E > PH * LD_WAVES)
#pragma unroll
            for (int u = PH; u < 2 * PH; ++u) pv[u] = rd(u);
    };
    pread(0);
    if (r1 < E) {
        const double Qb = (double)a.Qbar;
        auto g_of = [&](int m1, int k1, double qterm) {
            double v = s_v0[m1 * E + k1];
            if (a.Qbar > 0.0f) v += qterm;
            return v + s_nxt[m1 * E + k1];
        };
        double best = 0.0;
        if (a.pin && ((s_mask[r1] >> s) & 1u)) {
            best = g_of(s, r1, a.omega_Q * 0.0 / Qb);          // a local target is kept
        } else {
            bool have = false;
            // the target and its feasible substitutes (eq 7-8), budget-free
            while (kk[0] >= 0) {
                double qt[4];
                uint32_t srv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k1 = kk[u];
                    const bool on = k1 >= 0 && (k1 == r1 || sv[u] >= th);
                    const double q = k1 != r1 ? (double)((1.0f - sv[u]) * 0.5f) : 0.0;   // eq 18
                    qt[u] = a.omega_Q * q / Qb;
                    srv[u] = on ? s_mask[k1] : 0u;
                    if (a.allow_sub == 2 && k1 != r1) srv[u] &= 1u << s;   // local substitutes only
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    while (srv[u]) {
                        const int m1 = __builtin_ctz(srv[u]);
                        srv[u] &= srv[u] - 1;
                        const double v = g_of(m1, kk[u], qt[u]);
                        if (!have || v < best) { best = v; have = true; }
                    }
                }
                four();
            }
        }
        s_V[r1] = best;
    }
    __syncthreads();                                           // the costs are done with: s_P takes their place
    double acc = 0.0;
    static_assert(ORDERMOE_MAX_EXPERTS <= LD_THREADS, "one Phi entry per thread");
    for (int c0 = 0; c0 < E; c0 += LA_PC) {
        const int nc = E - c0 < LA_PC ? E - c0 : LA_PC;
        if (lane < nc) {
#pragma unroll
            for (int u = 0; u < PH; ++u)
                if (wave + u * LD_WAVES < E) s_P[(wave + u * LD_WAVES) * LA_LP + lane] = pv[u];
            if (E > PH * LD_WAVES)
#pragma unroll
                for (int u = PH; u < 2 * PH; ++u)
                    if (wave + u * LD_WAVES < E) s_P[(wave + u * LD_WAVES) * LA_LP + lane] = pv[u];
        }
        __syncthreads();
        pread(c0 + LA_PC);
        if (tid < E) {                                         // eq 42
            const double* pr = s_P + tid * LA_LP;
            const double* vr = s_V + c0;
            int c = 0;
            if (nc >= 16) {
                // the next eight columns are read while eight are summed
                f64x2 p0[4], v0[4], p1[4], v1[4];
                auto rd = [&](f64x2* p, f64x2* v, int at) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        p[u] = *(const f64x2*)(pr + at + 2 * u);
                        v[u] = *(const f64x2*)(vr + at + 2 * u);
                    }
                };
                auto add = [&](const f64x2* p, const f64x2* v) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) { acc += p[u][0] * v[u][0]; acc += p[u][1] * v[u][1]; }
                };
                rd(p0, v0, 0);
                for (; c + 16 <= nc; c += 16) {
                    rd(p1, v1, c + 8);
                    add(p0, v0);
                    rd(p0, v0, c + 16 <= nc - 8 ? c + 16 : 0);
                    add(p1, v1);
                }
            }
            for (; c < nc; ++c) acc += pr[c] * vr[c];
        }
        __syncthreads();
    }
    if (tid < E) out[tid] = acc;
}

unsigned blocks_for(int64_t n) {
    const int64_t b = (n + LA_THREADS - 1) / LA_THREADS;
    return (unsigned)(b < 1 ? 1 : (b > 65535 ? 65535 : b));
}

}  // namespace

size_t transitions_device_workspace(int32_t N, int32_t E) {
    return N > 1 ? (size_t)(N - 1) * E * E * sizeof(uint32_t) : 0;
}

size_t lookahead_device_workspace(int32_t N, int32_t E, int32_t M) {
    // the second Phi buffer of the ping-pong (the size allows two)
    return (size_t)2 * N * M * E * sizeof(double);
}

int launch_transitions_device(int32_t N, int32_t E, int64_t T_cal, const int32_t* top1, double* P, void* ws,
                              void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (N < 2) return 0;
    // Each block of the row kernel reads every token of its layer pair, with the
    // rows cut so that about 256 blocks run.  Its time grows with the tokens per
    // block, that of the device-memory counts with the tokens of all layers:
    // 128 experts, 32768 tokens: 18 against 45 us for 32 layers, 15.5 against
    // 13.7 us for 2; 2048 tokens: 8 against 18 us.
    if (T_cal <= TR_MAX_T) {
        int64_t R = ((int64_t)E * (N - 1) + 255) / 256;
        if (R > TR_LDS_COUNTS / E) R = TR_LDS_COUNTS / E;
        if (R > E) R = E;
        const int64_t nb = (E + R - 1) / R;
        transition_rows_kernel<<<dim3((unsigned)(nb * (N - 1))), LA_THREADS, 0, st>>>(top1, E, (int32_t)R, (int32_t)nb,
                                                                                      T_cal, P);
        return (int)hipGetLastError();
    }
    uint32_t* cnt = (uint32_t*)ws;
    const int64_t nc = (int64_t)(N - 1) * E * E;
    fill_u32<<<blocks_for(nc), LA_THREADS, 0, st>>>(cnt, nc);
    transition_count_kernel<<<blocks_for((int64_t)(N - 1) * T_cal), LA_THREADS, 0, st>>>(top1, N, E, T_cal, cnt);
    transition_norm_kernel<<<blocks_for((int64_t)(N - 1) * E * 64), LA_THREADS, 0, st>>>(cnt, N, E, P);
    return (int)hipGetLastError();
}

int launch_lookahead_device(const LookaheadDeviceArgs& d, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const int64_t ME = (int64_t)d.M * d.E, NME = (int64_t)d.N * ME;
    double* other = (double*)d.ws;                 // [N][M][E]
    if (d.H < 2 || d.N < 2) {
        fill_f64<<<blocks_for(NME), LA_THREADS, 0, st>>>(d.phi, NME);
        return (int)hipGetLastError();
    }
    LookArgs a;
    a.N = d.N; a.E = d.E; a.M = d.M; a.P = d.P; a.x = d.x; a.sim = d.sim; a.group_of = d.group_of;
    a.theta = d.theta; a.z_bits = d.z_bits; a.c = d.c; a.d_ref = d.d_ref; a.B = d.B; a.tau = d.tau;
    a.F = d.F; a.omega_T = d.omega_T; a.omega_Q = d.omega_Q; a.Qbar = d.Qbar; a.pin = d.pin;
    a.allow_sub = d.allow_sub;
    const size_t lds = lookahead_lds(d.E, d.M);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)lookahead_depth_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    // depth h writes the buffer that the last depth (H - 1) leaves in phi; depth 0 is zero
    const double* prev = nullptr;
    for (int h = 1; h <= d.H - 1; ++h) {
        double* cur = ((d.H - 1 - h) % 2 == 0) ? d.phi : other;
        lookahead_depth_kernel<<<dim3((unsigned)(((d.N + 7) / 8) * 8 * d.M)), LD_THREADS, lds, st>>>(a, prev, cur);
        prev = cur;
    }
    return (int)hipGetLastError();
}

}  // namespace ordermoe
