// Fully connected products on the bf16 matrix instructions with FP32 operands held whole (the operands,
// part products and sign changes are those of conv_split.hip): back-substitution C = A W (Eq. 2) and the
// adjoint's forward product C = G W^T + b.
//
// The reduction of a layer is cut into KP parts of consecutive 32-term steps (one, four or eight by its
// length alone); each part has its own accumulators and the parts' sums are added in order.  So the two
// kernels below give the same bits, and a row's result does not depend on the batch:
//
// k_fc_tile, for many rows: 128 rows x 128 outputs per workgroup of eight wavefronts, the parts one after
// the other.  The rows are cut into parts once per workgroup and step on their way into LDS (a row's
// eight terms and three parts in 48 consecutive bytes, double-buffered); the filters come from their
// stream, laid out in the order the wavefronts read it.  The cutting is as long as the matrix work that
// follows from it, so it has no branch and its instructions are interleaved with the matrix ones; octets that
// need the branch (infinities, values that round up to one) are cut again behind them.
// 9216 rows of 4096 -> 512 back: 250 us (155 TFLOP/s), 391 us on the FP32 instructions before.
//
// k_fc_parts, for few: a wavefront per part and 16 rows x 32 outputs per workgroup, operands straight
// into registers, one exchange through LDS at the end.  A layer of few rows was a chain of K / 16 loads
// and barriers on a handful of workgroups: 9 rows of 784 -> 100 took 42 us and take 8, 4096 -> 512 206 us
// and 16.
#include "kernels.h"
#include "split.h"

namespace mnb {
namespace {

struct FcArgs {
    const float* A; float* C; const unsigned char* Ws; const float* bias;
    int M, N, K, nk, parts;
    int acc, vec_in, vec_out;
    int mb, nb;      // row and output blocks of the tile kernel
};

constexpr int BM = 128, BN = 128, FM = 4, FN = 2;   // eight wavefronts of 64 rows x 32 outputs
constexpr int PLANE = BM * POSB + 64;               // bytes of one octet of a step's 32 terms
constexpr int BUF = 4 * PLANE;

__device__ __forceinline__ int part_begin(const FcArgs& a, int p) { return (int)((long)a.nk * p / a.parts); }

// eight consecutive terms of row r (addresses clamped to the rows: row M - 1 stands in for rows past the
// end; terms beyond K are masked where they are used, so that nothing waits for the loads here)
__device__ __forceinline__ void load8(const FcArgs& a, int r, int k, float* x) {
    const float* s = a.A + (long)min(r, a.M - 1) * a.K;
    if (a.vec_in) {   // K a multiple of 4, aligned
        const floatx4 v = *reinterpret_cast<const floatx4*>(s + min(k, a.K - 4));
        const floatx4 w = *reinterpret_cast<const floatx4*>(s + min(k + 4, a.K - 4));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = v[i];
            x[4 + i] = w[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = s[min(k + i, a.K - 1)];
    }
}
// step k's terms beyond K to zero
__device__ __forceinline__ void mask8(const FcArgs& a, int step, int k, float* x) {
    if (step * 32 + 32 <= a.K) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = k + i < a.K ? x[i] : 0.f;
}

// one fragment's results: row r, outputs n .. n + 3
__device__ __forceinline__ void store4(const FcArgs& a, int r, int n, floatx4 t) {
    if (r >= a.M) return;
    float* o = a.C + (long)r * a.N + n;
    if (a.vec_out && n < a.N) {
        if (a.bias) t += *reinterpret_cast<const floatx4*>(a.bias + n);
        if (a.acc) t += *reinterpret_cast<floatx4*>(o);
        *reinterpret_cast<floatx4*>(o) = t;
        return;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (n + v >= a.N) continue;
        float s = t[v] + (a.bias ? a.bias[n + v] : 0.f);
        if (a.acc) s += o[v];
        o[v] = s;
    }
}

__global__ __launch_bounds__(512, 2) void k_fc_tile(FcArgs a) {
    extern __shared__ unsigned char sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups go to the eight dies in turn: each die keeps every eighth row block, whose rows stay in
    // its L2 while it goes through the outputs
    const int die = blockIdx.x & 7, idx = blockIdx.x >> 3, per = (a.mb + 7) / 8;
    const int mi = die + 8 * (idx % per), ni = idx / per;
    if (mi >= a.mb) return;
    const int m0 = mi * BM, n0 = ni * BN;
    const int wm = wave & 1, wn = wave >> 1;
    const int ntiles = (a.N + 15) / 16, t0 = n0 / 16 + wn * FN;
    const unsigned char* wp[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) wp[j] = a.Ws + (long)min(t0 + j, ntiles - 1) * a.nk * STEPB;
    const int lo16 = lane * 16;

    // this thread's octet of a step: row sr, terms 8 sk .. 8 sk + 7
    const int sr = tid >> 2, sk = tid & 3;
    const int dst = sk * PLANE + sr * POSB;
    float x[2][8];   // the next step's octet and the one after it
    auto put = [&](int b, uintx4 p0, uintx4 p1, uintx4 p2) {
        unsigned char* d = sm + b * BUF + dst;
        *reinterpret_cast<uintx4*>(d) = p0;
        *reinterpret_cast<uintx4*>(d + 16) = p1;
        *reinterpret_cast<uintx4*>(d + 32) = p2;
    };
    uintx4 p0, p1, p2;
    load8(a, m0 + sr, sk * 8, x[0]);
    bf16x8 wb[2][FN][3];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int s = 0; s < 3; ++s) wb[0][j][s] = *reinterpret_cast<const bf16x8*>(wp[j] + s * 1024 + lo16);
    load8(a, m0 + sr, 32 + sk * 8, x[1]);
    mask8(a, 0, sk * 8, x[0]);
    mask8(a, 1, 32 + sk * 8, x[1]);
    split8(x[0], p0, p1, p2);
    put(0, p0, p1, p2);
    __syncthreads();

    floatx4 hi[FN][FM], low[FN][FM], sum[FN][FM];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i) hi[j][i] = low[j][i] = sum[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int rb = (lane >> 4) * PLANE + (wm * FM * 16 + (lane & 15)) * POSB;
    int part = 0, begin = 0, end = part_begin(a, 1), half = begin + (end - begin + 1) / 2;
    // Step k (b = k & 1): reads issued for the filters one step and the rows two steps ahead (in this order,
    // so that waiting for the filters does not wait for the rows), then the next step's rows cut and
    // written beside this step's matrix instructions.
    auto step = [&](int k, int b) {
        const unsigned char* buf = sm + b * BUF + rb;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int s = 0; s < 3; ++s)
                wb[b ^ 1][j][s] = *reinterpret_cast<const bf16x8*>(wp[j] + (long)(k + 1) * STEPB + s * 1024 + lo16);
        load8(a, m0 + sr, (k + 2) * 32 + sk * 8, x[b]);
        bf16x8 rf[FM][3];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int s = 0; s < 3; ++s) rf[i][s] = *reinterpret_cast<const bf16x8*>(buf + i * 16 * POSB + s * 16);
        split8<false>(x[b ^ 1], p0, p1, p2);
        put(b ^ 1, p0, p1, p2);
        const float big = max8(x[b ^ 1]);
#pragma unroll
        for (int i = 0; i < FM; ++i) MNB_SPLIT_MM(FN, wb[b], rf[i], hi, low, i)
        // one matrix instruction, then up to two vector ones in its shadow (three: 1 to 3 % slower)
#pragma unroll
        for (int q = 0; q < 48; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        }
        if (big >= SPLIT_BIG) {   // cut again, where it is not among the matrix instructions
            split8(x[b ^ 1], p0, p1, p2);
            put(b ^ 1, p0, p1, p2);
        }
        mask8(a, k + 2, (k + 2) * 32 + sk * 8, x[b]);   // (waits for the rows only where K ends)
        if (k + 1 == half) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    hi[j][i] = -hi[j][i];
                    low[j][i] = -low[j][i];
                }
        }
        if (k + 1 == end) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    sum[j][i] -= hi[j][i] + low[j][i];
                    hi[j][i] = low[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            ++part;
            begin = end;
            end = part_begin(a, part + 1);
            half = begin + (end - begin + 1) / 2;
        }
        __syncthreads();
    };
    for (int k = 0; k < a.nk; k += 2) {
        step(k, 0);
        if (k + 1 < a.nk) step(k + 1, 1);
    }
    // result lanes: row lane % 16 of fragment i, outputs 4 (lane / 16) + v of fragment j
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
            store4(a, m0 + (wm * FM + i) * 16 + (lane & 15), n0 + (wn * FN + j) * 16 + 4 * (lane >> 4), sum[j][i]);
}

template <int KP>
__global__ __launch_bounds__(64 * KP) void k_fc_parts(FcArgs a) {
    __shared__ floatx4 ex[KP][2][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.x * 16, t0 = blockIdx.y * 2;
    const int ntiles = (a.N + 15) / 16;
    const unsigned char* wp[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) wp[j] = a.Ws + (long)min(t0 + j, ntiles - 1) * a.nk * STEPB + lane * 16;
    const int r = m0 + (lane & 15), k8 = (lane >> 4) * 8;
    const int begin = part_begin(a, wave), end = part_begin(a, wave + 1), half = begin + (end - begin + 1) / 2;
    floatx4 hi[2][1], low[2][1];
#pragma unroll
    for (int j = 0; j < 2; ++j) hi[j][0] = low[j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
    // four steps' operands in flight
    constexpr int D = 4;
    float x[D][8];
    bf16x8 w[D][2][3];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int k = min(begin + d, a.nk - 1);
        load8(a, r, k * 32 + k8, x[d]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int s = 0; s < 3; ++s) w[d][j][s] = *reinterpret_cast<const bf16x8*>(wp[j] + (long)k * STEPB + s * 1024);
    }
    for (int k0 = begin; k0 < end; k0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int k = k0 + d;
            if (k >= end) break;
            mask8(a, k, k * 32 + k8, x[d]);
            uintx4 p0, p1, p2;
            split8(x[d], p0, p1, p2);
            const bf16x8 rf[3] = {__builtin_bit_cast(bf16x8, p0), __builtin_bit_cast(bf16x8, p1),
                                  __builtin_bit_cast(bf16x8, p2)};
            MNB_SPLIT_MM(2, w[d], rf, hi, low, 0)
            if (k + 1 == half) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    hi[j][0] = -hi[j][0];
                    low[j][0] = -low[j][0];
                }
            }
            const int kn = min(k + D, a.nk - 1);
            load8(a, r, kn * 32 + k8, x[d]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int s = 0; s < 3; ++s)
                    w[d][j][s] = *reinterpret_cast<const bf16x8*>(wp[j] + (long)kn * STEPB + s * 1024);
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) ex[wave][j][lane] = hi[j][0] + low[j][0];
    __syncthreads();
    if (wave >= 2 || (KP == 1 && wave > 0)) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (KP > 1 && wave != j) continue;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < KP; ++p) sum -= ex[p][j][lane];
        if (t0 + j < ntiles) store4(a, r, (t0 + j) * 16 + 4 * (lane >> 4), sum);
    }
}

struct FcStream {
    const float* W; unsigned short* out;
    int N, K, nk, parts, back;
};
__global__ __launch_bounds__(256) void k_fc_stream(FcStream a, long n) {
    const long id = (long)blockIdx.x * 256 + threadIdx.x;
    if (id >= n) return;
    const int j = (int)(id & 7), lane = (int)(id >> 3) & 63;
    const long rest = id >> 9;   // tile * nk + step
    const int k = (int)(rest % a.nk), nt = (int)(rest / a.nk);
    const int o = nt * 16 + (lane & 15), kk = k * 32 + (lane >> 4) * 8 + j;
    int p = 0;
    while (k >= (int)((long)a.nk * (p + 1) / a.parts)) ++p;
    const int begin = (int)((long)a.nk * p / a.parts), end = (int)((long)a.nk * (p + 1) / a.parts);
    float w = 0.f;
    if (o < a.N && kk < a.K) {
        w = a.back ? a.W[(long)kk * a.N + o] : a.W[(long)o * a.K + kk];
        if (k >= begin + (end - begin + 1) / 2) w = -w;
    }
    split_weight(w, a.out + rest * (STEPB / 2) + lane * 8 + j);
}

int fc_parts(int nk) { return nk >= 64 ? 8 : nk >= 8 ? 4 : 1; }

void launch_fc(const unsigned char* Ws, const float* A, const float* bias, float* C, int M, int N, int K, bool accumulate,
               hipStream_t st) {
    FcArgs a{};
    a.A = A; a.C = C; a.Ws = Ws; a.bias = bias;
    a.M = M; a.N = N; a.K = K; a.nk = cdiv(K, 32); a.parts = fc_parts(a.nk);
    a.acc = accumulate;
    a.vec_in = K % 4 == 0 && ((uintptr_t)A & 15) == 0;
    a.vec_out = N % 4 == 0 && ((uintptr_t)C & 15) == 0 && (!bias || ((uintptr_t)bias & 15) == 0);
    a.mb = cdiv(M, BM);
    a.nb = cdiv(N, BN);
    // A tile takes about 1.4 us a step however few there are (up to one per compute unit), a 16 x 32 block
    // of the other kernel its share of the chip, 0.6 ns a step: equal near 72 tiles.  100, 500 and 1024
    // rows of 512 -> 4096 (32, 128, 256 tiles): 24, 63 and 119 us in blocks, 34, 35 and 36 in tiles; 1024,
    // 2048 and 4096 rows of 4096 -> 512 (32, 64, 128): 78, 150 and 300 against 181
    const long tiles = (long)a.mb * a.nb;
    if (tiles >= 72) {
        const long grid = 8l * cdiv(a.mb, 8) * a.nb;
        MNB_CHECK(grid <= 0x7fffffffL, -2, "too many rows for one product");
        hipLaunchKernelGGL(k_fc_tile, dim3((unsigned)grid), dim3(512), 2 * BUF, st, a);
    } else {
        const dim3 grid(cdiv(M, 16), cdiv(N, 32));
        if (a.parts == 8) hipLaunchKernelGGL(k_fc_parts<8>, grid, dim3(512), 0, st, a);
        else if (a.parts == 4) hipLaunchKernelGGL(k_fc_parts<4>, grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(k_fc_parts<1>, grid, dim3(64), 0, st, a);
    }
    MNB_HIP(hipGetLastError());
}

}  // namespace

size_t fc_stream_bytes(int N, int K) { return ((size_t)cdiv(N, 16) * cdiv(K, 32) + 1) * STEPB; }

void launch_fc_stream(const float* W, int N, int K, bool back, void* out, hipStream_t st) {
    FcStream s{W, (unsigned short*)out, N, K, cdiv(K, 32), fc_parts(cdiv(K, 32)), back};
    const long n = (long)cdiv(N, 16) * s.nk * 512;
    hipLaunchKernelGGL(k_fc_stream, dim3(cdiv(n, 256)), dim3(256), 0, st, s, n);
    MNB_HIP(hipGetLastError());
}

void launch_fc_backsub(const unsigned char* Ws, const float* A, float* C, int M, int dout, int din, bool accumulate,
                       hipStream_t st) {
    if (M > 0) launch_fc(Ws, A, nullptr, C, M, din, dout, accumulate, st);
}
void launch_fc_forward(const unsigned char* Ws, const float* G, const float* b, float* C, int M, int din, int dout,
                       bool accumulate, hipStream_t st) {
    if (M > 0) launch_fc(Ws, G, b, C, M, dout, din, accumulate, st);
}

}  // namespace mnb
