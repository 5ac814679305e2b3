// Convolutions on the bf16 matrix instructions with FP32 operands held whole: the forward product of
// the adjoint and the transposed convolution of back-substitution (Eq. 2), from input windows staged in
// LDS.
//
// Operands.  Each FP32 value is cut into three bf16 parts that add up to it (from 2^-110 on; below, to
// 2^-134), x = x0 + x1 + x2, each the nearest to what is left, and a product is the sum of the six part
// products x_i w_j with i + j <= 2, accumulated in FP32 by v_mfma_f32_16x16x32_bf16.  x1 and w1 are at most
// 2^-8, x2 and w2 2^-17 of their value's leading power of two, so the three products left out are at most
// 2^-24 + 2^-34 of the product (2^-27.4 in the mean square of 4e6 random pairs) and have no preferred sign.
// That shows in a sum of one term alone, off by up to 1.0e-7 (2.6e-8 in the mean square) where FP32's
// rounding is by 6.0e-8 (2.5e-8); with weights cut off instead of rounded it was 2.0e-7 (3.1e-8).
// Six instructions of 16 cycles for 32 terms of a 16x16 tile take 96 cycles where the FP32 instruction
// takes 256, so the FP32 matrix rate (154 TFLOP/s measured) no longer bounds the layer: the bf16
// instruction sustains 2.0 PFLOP/s, 333 TFLOP/s of such products.  The activations are cut while they
// are staged, the filters once, when the net is created.
//
// Rounding.  The instruction adds groups of eight products with the lower bits of the smaller ones cut
// off downwards: every sum of the leading products comes out a little low (1e-8 of its terms), the same
// way for every output, and over the inputs of a network that adds up (the bounds of ConvBig's fourth
// layer moved by 1.5e-6, seven times their FP32 error).  So the accumulators change sign half way
// through each stage and the filters of the second half enter negated: the two halves' errors cancel.
// The five small part products have accumulators of their own, added at the end, so that they do not
// round the large sum once more each.  Error of a layer against FP64: 7.6e-8, 1.1e-7 and 5.6e-8 back
// through ConvBig's three layers, where the FP32 instructions give 2.1e-7, 3.2e-7 and 1.4e-7 (mean of the
// errors 1e-10 of the values in both); of the fourth layer's bounds 2.0e-7 against 2.3e-7.
//
// Infinities and NaN give what FP32 products give (see split8); so does a product beyond FP32's range, or
// NaN from 2^8 times it on, where the small part products leave it too.
//
// Work split.  One workgroup owns BM output positions (part of a row's grid, or the whole grids of R
// rows) and BN filters.  Per stage of CGS 8-channel groups it writes the input window those positions
// read into LDS, channel-last, a position's eight channels and three parts in 48 consecutive bytes: a
// fragment's 16 positions then lie in distinct banks at stride 1 and 2 alike (121 of 128 bytes a cycle
// measured).  A reduction step is 32 terms: four channel groups of one filter tap, or fewer groups of
// two or four neighbouring taps.  The filters are not staged: their stream, cut and laid out in the order
// the wavefronts use it, comes from the caches (16 bytes a lane, one step ahead).  A transposed stride-2
// convolution computes its four output phases in one workgroup; phases that read the same window
// column share its fragment.
//
// An output sums its stages, window offsets and part products in an order fixed by the layer, whatever
// the batch and tile: a row's result does not depend on the rows around it.
//
// What bounds it, by its counters: the matrix units are busy 38 to 59 % of the time; the rest is the cutting
// and writing of the window between two barriers and, at 4x4 / 2, the wait for the input itself.  2048
// rows of 32x16x16 -> 64 (3x3) take 100 us (190 TFLOP/s; 207 us on the FP32 instructions before); without
// its global loads and stores the kernel takes 75 us, with them alone 40.  32x32x32 -> 32x16x16 (4x4 / 2):
// 125 us against 203 before at 2.7 TB/s, back 142 us against 225.
#include "kernels.h"
#include "split.h"
#include "../../include/mnbab.h"

namespace mnb {
namespace {

constexpr size_t SPLIT_LDS_MAX = 64 * 1024;    // of a workgroup's window
constexpr size_t SPLIT_LDS_ROWS = 40 * 1024;   // ... while it takes several rows: four workgroups a CU

struct SplitArgs {
    const float* G; float* C; const unsigned char* Ws; const float* bias;
    long ldG, ldC;
    int M, Hi, Wi, Co, Ho, Wo, p;      // input plane, output grid of a phase, padding of window row/col 0
    int R, mtiles, P, ng, acc;          // rows per workgroup, tiles per row (R == 1), positions, stages
    int WH, RS, plane;                  // window rows per row, row stride, positions per channel group
    int oH, oW, out_s;                  // output plane and stride of the grid on it
    ConeClip clip;
    float rWo, rP, rWi;
    bool quad;      // the stores of consecutive outputs are aligned (16 bytes, phases: 8 bytes)
};

__device__ __forceinline__ int qdiv(int i, float r) { return (int)(((float)i + 0.5f) * r); }

// Whether position pos of row r lies outside the node of a cone row.
__device__ __forceinline__ bool clipped(const SplitArgs& a, int r, int pos) {
    int oy, ox;
    cone_origin(a.clip, r, oy, ox);
    const int y = qdiv(pos, a.rWo), x = pos - y * a.Wo;
    return !(oy + y >= 0 && oy + y < a.clip.H && ox + x >= 0 && ox + x < a.clip.W);
}
__device__ __forceinline__ void clip_quad(const SplitArgs& a, int r, int pos, bool* zero) {
    int oy, ox;
    cone_origin(a.clip, r, oy, ox);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int y = qdiv(pos + v, a.rWo), x = pos + v - y * a.Wo;
        zero[v] = !(oy + y >= 0 && oy + y < a.clip.H && ox + x >= 0 && ox + x < a.clip.W);
    }
}

// One dimension's pattern: phase a reads window offsets O[a] .. O[a] + N[a] - 1.
template <int O0, int N0, int O1, int N1>
struct Pat {
    __host__ __device__ static constexpr int off(int a) { return a ? O1 : O0; }
    __host__ __device__ static constexpr int cnt(int a) { return a ? N1 : N0; }
    __host__ __device__ static constexpr int nd() { return (O0 + N0) > (O1 + N1) ? (O0 + N0) : (O1 + N1); }
};

// Whether phase (pa, pb) has a reduction step at window row oy over the columns xs .. xs + rem - 1.
template <class PT, int UT>
__host__ __device__ constexpr bool uses(int pa, int pb, int oy, int xs, int rem) {
    return oy >= PT::off(pa) && oy < PT::off(pa) + PT::cnt(pa) && xs >= PT::off(pb) &&
           xs < PT::off(pb) + PT::cnt(pb) && (xs - PT::off(pb)) % UT == 0 &&
           (PT::off(pb) + PT::cnt(pb) - xs < UT ? PT::off(pb) + PT::cnt(pb) - xs : UT) == rem;
}

// A stage's reduction steps: window offset, lanes in use, phase, and the number of the fragment set
// (steps of several phases at one offset share it).
template <class PT, int NP, int UT>
struct StepTable {
    static constexpr int MAX = PT::nd() * PT::nd() * NP * NP;
    int n = 0;
    int oy[MAX]{}, xs[MAX]{}, rem[MAX]{}, ph[MAX]{}, set[MAX]{};
    bool late[MAX]{}, flip[MAX]{};   // in the second half of its phase's steps, the last one of the first
    __host__ __device__ constexpr StepTable() {
        int sets = 0;
        for (int y = 0; y < PT::nd(); ++y)
            for (int xr = 0; xr < PT::nd() * UT; ++xr) {
                bool any = false;
                for (int f = 0; f < NP * NP; ++f)
                    if (uses<PT, UT>(f / NP, f % NP, y, xr / UT, UT - xr % UT)) {
                        oy[n] = y; xs[n] = xr / UT; rem[n] = UT - xr % UT; ph[n] = f; set[n] = sets;
                        ++n;
                        any = true;
                    }
                if (any) ++sets;
            }
        for (int f = 0; f < NP * NP; ++f) {
            int count = 0, at = 0;
            for (int t = 0; t < n; ++t) count += ph[t] == f;
            for (int t = 0; t < n; ++t) {
                if (ph[t] != f) continue;
                late[t] = at >= (count + 1) / 2;
                flip[t] = ++at == (count + 1) / 2;
            }
        }
    }
};

template <class PT, int NP, int S, int CGS, int FN, int FM, int WN, int WM>
__global__ __launch_bounds__(64 * WN * WM, (FN * FM * NP >= 8 ? 2 : 3)) void k_conv_split(SplitArgs a) {
    constexpr int NT = 64 * WN * WM, UT = 4 / CGS, BM = 16 * FM * WM;
    // Whether the next step's reads are held ahead of this step's matrix instructions (left to itself the
    // compiler moves them down to their use, which needs fewer registers).  Ahead against not, TFLOP/s:
    // 3x3 / 1 with two position fragments a wavefront 173 / 157 (16x16 -> 32), 170 / 163 (8x8), with four
    // 186 / 193; 4x4 / 2 into 64 channels 187 / 177, into 32 127 / 127; 3x3 / 2 114 / 108 and 89 / 91;
    // transposed 4x4 / 2 115 / 120, 121 / 95, 156 / 133, transposed 3x3 / 2 91 / 98
    constexpr bool AHEAD = NP == 2 ? PT::cnt(0) == 2 && PT::cnt(1) == 2
                           : S == 1 ? FM <= 2 : PT::cnt(0) > 1 && (FN * WN >= 4 || (PT::cnt(0) == 4 && FN == 2 && FM == 4));
    extern __shared__ unsigned char sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    int r0, m0, y_first, rows;
    if (a.R > 1) {
        r0 = blockIdx.x * a.R; m0 = 0; y_first = 0;
        rows = min(a.R, a.M - r0);
    } else {
        r0 = blockIdx.x / a.mtiles; m0 = (blockIdx.x - r0 * a.mtiles) * BM;
        y_first = __builtin_amdgcn_readfirstlane(qdiv(m0, a.rWo));
        rows = 1;
    }
    const int n0 = blockIdx.y * (16 * FN * WN);
    const int iy0 = S * y_first - a.p;
    const int wy_lo = max(0, -iy0), wy_hi = min(a.WH, a.Hi - iy0);
    const int nvr = max(0, wy_hi - wy_lo);
    const int HiWi = a.Hi * a.Wi;
    const int per_c = nvr * a.Wi, per_r = CGS * per_c, total = rows * per_r;
    const float rpc = 1.f / (float)max(per_c, 1), rpr = 1.f / (float)max(per_r, 1);

    // zero the window once: padding and positions outside the plane are never written again
    for (int i = tid; i < (CGS * a.plane + 1) * (POSB / 16); i += NT)
        *reinterpret_cast<uintx4*>(sm + i * 16) = uintx4{0, 0, 0, 0};

    // lane bases of the position fragments
    int xb[FM];
    const int cgl = (lane >> 4) % CGS, ux = (lane >> 4) / CGS;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int q = (wm * FM + i) * 16 + (lane & 15);
        int rl = 0, pos = m0 + q;
        if (a.R > 1) { rl = qdiv(q, a.rP); pos = q - rl * a.P; }
        int w = cgl * a.plane + ux;
        if (rl < rows && pos < a.P) {
            const int y = qdiv(pos, a.rWo), x = pos - y * a.Wo;
            w += (rl * a.WH + S * (y - y_first)) * a.RS + S * x;
        }
        xb[i] = w * POSB;
    }
    const int zero_at = CGS * a.plane * POSB;

    floatx4 acc[NP * NP][FN][FM], low[NP * NP][FN][FM];
#pragma unroll
    for (int f = 0; f < NP * NP; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) acc[f][j][i] = low[f][j][i] = floatx4{0.f, 0.f, 0.f, 0.f};

    // reduction steps of a stage
    constexpr int NSTEP = StepTable<PT, NP, UT>{}.n;
    const long stream = (long)a.ng * NSTEP * STEPB;
    const unsigned char* wp[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) wp[j] = a.Ws + (long)(n0 / 16 + wn * FN + j) * stream;
    const int lo16 = lane * 16;

    bf16x8 ab[2][FN][3];
#define MNB_LOADA(buf, at)                                                                   \
    _Pragma("unroll") for (int j = 0; j < FN; ++j) _Pragma("unroll") for (int s = 0; s < 3; ++s) \
        ab[buf][j][s] = *reinterpret_cast<const bf16x8*>(wp[j] + (at) + s * 1024 + lo16);
    MNB_LOADA(0, 0L)

    for (int g = 0; g < a.ng; ++g) {
        __syncthreads();   // previous stage consumed (or the zero fill done)
        // one base address per channel of a group and a 32-bit offset per thread, shared by the eight loads
        const char* src = reinterpret_cast<const char*>(a.G + (long)r0 * a.ldG + (long)g * (CGS * 8) * HiWi +
                                                        (long)(iy0 + wy_lo) * a.Wi);
        for (int e0 = tid; e0 < total; e0 += 2 * NT) {
            float x[2][8];
            int dst[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e = min(e0 + h * NT, total - 1);
                const int rl = a.R > 1 ? qdiv(e, rpr) : 0;
                const int er = e - rl * per_r;
                const int c = CGS > 1 ? qdiv(er, rpc) : 0;
                const int rem = er - c * per_c;
                const int row = qdiv(rem, a.rWi), col = rem - row * a.Wi;
                const unsigned at = (unsigned)(rl * (int)a.ldG + c * 8 * HiWi + rem) * 4u;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    x[h][k] = *reinterpret_cast<const float*>(src + (long)k * HiWi * 4 + at);
                dst[h] = (c * a.plane + (rl * a.WH + wy_lo + row) * a.RS + a.p + col) * POSB;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && e0 + NT >= total) break;
                uintx4 p0, p1, p2;
                split8(x[h], p0, p1, p2);
                *reinterpret_cast<uintx4*>(sm + dst[h]) = p0;
                *reinterpret_cast<uintx4*>(sm + dst[h] + 16) = p1;
                *reinterpret_cast<uintx4*>(sm + dst[h] + 32) = p2;
            }
        }
        __syncthreads();
        // Steps in order; step t's window fragments sit in buffer (its fragment set's number) & 1 and its
        // filters in buffer t & 1.  A step first issues the reads of the next one.
        bf16x8 bf[2][FM][3];
        constexpr StepTable<PT, NP, UT> T{};
#define MNB_LOADB(buf, t_)                                                                             \
    _Pragma("unroll") for (int i = 0; i < FM; ++i) {                                                   \
        int ad_ = xb[i] + (T.oy[t_] * a.RS + T.xs[t_]) * POSB;                                         \
        if (T.rem[t_] < UT && ux >= T.rem[t_]) ad_ = zero_at;                                          \
        _Pragma("unroll") for (int s = 0; s < 3; ++s)                                                  \
            bf[buf][i][s] = *reinterpret_cast<const bf16x8*>(sm + ad_ + s * 16);                       \
    }
        MNB_LOADB(0, 0)
#pragma unroll
        for (int t = 0; t < NSTEP; ++t) {
            MNB_LOADA((t + 1) & 1, (long)(g * NSTEP + t + 1) * STEPB)
            const int cb = T.set[t] & 1, cu = t & 1, f = T.ph[t];
            if (t + 1 < NSTEP && T.set[t + 1] != T.set[t]) { MNB_LOADB(T.set[t + 1] & 1, t + 1) }
            if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
#define MNB_MM(to, sa, sb)                                                                           \
    _Pragma("unroll") for (int j = 0; j < FN; ++j) _Pragma("unroll") for (int i = 0; i < FM; ++i)     \
        to[f][j][i] = NP == 1 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[cb][i][sb], ab[cu][j][sa], to[f][j][i], 0, 0, 0) \
                                   : __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab[cu][j][sa], bf[cb][i][sb], to[f][j][i], 0, 0, 0);
            MNB_MM(low, 2, 0) MNB_MM(acc, 0, 0) MNB_MM(low, 1, 1) MNB_MM(low, 0, 2) MNB_MM(low, 1, 0) MNB_MM(low, 0, 1)
            if (T.flip[t]) {
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i) {
                        acc[f][j][i] = -acc[f][j][i];
                        low[f][j][i] = -low[f][j][i];
                    }
            }
            if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
        if (NSTEP & 1) {   // the next stage starts on buffer 0
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int s = 0; s < 3; ++s) ab[0][j][s] = ab[1][j][s];
        }
    }
#undef MNB_LOADA
#undef MNB_LOADB
#undef MNB_MM

    const int oHW = a.oH * a.oW;
#pragma unroll
    for (int f = 0; f < NP * NP; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) acc[f][j][i] += low[f][j][i];
    if constexpr (NP == 1) {
        // result lanes: filter 16 j + lane % 16, positions 4 (lane / 16) + v of fragment i, which go
        // out as one 16-byte store where they are consecutive and aligned
        float* Cl = a.C + (long)(n0 + wn * FN * 16 + (lane & 15)) * oHW;
        float bias[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) bias[j] = a.bias ? a.bias[n0 + (wn * FN + j) * 16 + (lane & 15)] : 0.f;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int q = (wm * FM + i) * 16 + 4 * (lane >> 4);
            int rl = 0, pos = m0 + q;
            if (a.R > 1) { rl = qdiv(q, a.rP); pos = q - rl * a.P; }
            if (a.quad) {
                if (rl >= rows || pos >= a.P) continue;
                bool zero[4] = {false, false, false, false};
                if (a.clip.rows) clip_quad(a, r0 + rl, pos, zero);
                float* o = Cl + (long)(r0 + rl) * a.ldC + pos;
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    floatx4 t;
#pragma unroll
                    for (int v = 0; v < 4; ++v) t[v] = zero[v] ? 0.f : acc[0][j][i][v] + bias[j];
                    floatx4* o4 = reinterpret_cast<floatx4*>(o + (long)j * 16 * oHW);
                    if (a.acc) t += *o4;
                    *o4 = t;
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int rv = rl, pv = pos + v;
                    if (a.R > 1) {   // (on a grid of one position the four belong to four rows)
                        rv = qdiv(q + v, a.rP);
                        pv = q + v - rv * a.P;
                    }
                    if (rv >= rows || pv >= a.P) continue;
                    bool zero = false;
                    if (a.clip.rows) zero = clipped(a, r0 + rv, pv);
                    float* o = Cl + (long)(r0 + rv) * a.ldC + pv;
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        float t = zero ? 0.f : acc[0][j][i][v] + bias[j];
                        float* o1 = o + (long)j * 16 * oHW;
                        if (a.acc) t += *o1;
                        *o1 = t;
                    }
                }
            }
        }
    } else {
        // result lanes: position lane % 16 of fragment i, filters 16 j + 4 (lane / 16) + v; a
        // position's two column phases are neighbours on the output
        float* Cl = a.C + (long)(n0 + wn * FN * 16 + 4 * (lane >> 4)) * oHW;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int q = (wm * FM + i) * 16 + (lane & 15);
            int rl = 0, pos = m0 + q;
            if (a.R > 1) { rl = qdiv(q, a.rP); pos = q - rl * a.P; }
            if (rl >= rows || pos >= a.P) continue;
            const int y = qdiv(pos, a.rWo), x = pos - y * a.Wo;
            const int X = 2 * x;
            const bool two = X + 1 < a.oW;
#pragma unroll
            for (int pa = 0; pa < 2; ++pa) {
                const int Y = 2 * y + pa;
                if (Y >= a.oH || X >= a.oW) continue;
                float* o = Cl + (long)(r0 + rl) * a.ldC + Y * a.oW + X;
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float* o2 = o + (long)(j * 16 + v) * oHW;
                        floatx2 t = {acc[pa * 2][j][i][v], acc[pa * 2 + 1][j][i][v]};
                        if (a.quad) {
                            if (a.acc) t += *reinterpret_cast<floatx2*>(o2);
                            *reinterpret_cast<floatx2*>(o2) = t;
                        } else {
                            o2[0] = a.acc ? o2[0] + t[0] : t[0];
                            if (two) o2[1] = a.acc ? o2[1] + t[1] : t[1];
                        }
                    }
            }
        }
    }
}


// ------------------------------------------------------------------ filter streams
// Steps of a stage: step t's octet-column u holds tap (ky, kx) of the filter (tap[t * UT + u] =
// ky << 8 | kx, -1: none).
struct StreamArgs {
    const float* W; unsigned short* out;
    int Cin, Cout, k, back, ng, cgs, nstep;
    short tap[64];
    unsigned long long late;   // steps whose filters enter with the opposite sign
};

__global__ __launch_bounds__(256) void k_split_stream(StreamArgs a, long n) {
    const long id = (long)blockIdx.x * 256 + threadIdx.x;
    if (id >= n) return;
    const int j = (int)(id & 7), lane = (int)(id >> 3) & 63;
    const long rest = id >> 9;                       // ((nt * ng + g) * nstep + t)
    const int t = (int)(rest % a.nstep);
    const int g = (int)(rest / a.nstep % a.ng), nt = (int)(rest / a.nstep / a.ng);
    const int f = nt * 16 + (lane & 15), c = (g * a.cgs + (lane >> 4) % a.cgs) * 8 + j;
    const int tap = a.tap[t * (4 / a.cgs) + (lane >> 4) / a.cgs];
    float w = 0.f;
    if (tap >= 0 && f < a.Cout && c < a.Cin) {
        const long o = a.back ? (long)c * a.Cout + f : (long)f * a.Cin + c;
        w = a.W[(o * a.k + (tap >> 8)) * a.k + (tap & 255)];
        // the accumulators change sign once a stage, and end with the sign of the sum
        if (((a.ng - g) & 1) != (int)(a.late >> t & 1)) w = -w;
    }
    unsigned short* dst = a.out + rest * (STEPB / 2) + lane * 8 + j;
    split_weight(w, dst);
}

enum { PAT_F31, PAT_F21, PAT_F42, PAT_F32, PAT_F12, PAT_T42D, PAT_T42S, PAT_T32D, PAT_T32S, PAT_T12 };
typedef Pat<0, 3, 0, 0> P3;
typedef Pat<0, 4, 0, 0> P4;
typedef Pat<0, 2, 0, 0> P2;
typedef Pat<0, 1, 0, 0> P1;
typedef Pat<0, 2, 1, 2> P42D;
typedef Pat<0, 2, 0, 2> P42S;
typedef Pat<0, 1, 0, 2> P32D;
typedef Pat<0, 2, 1, 1> P32S;

template <class PT, int NP, int UT, class F>
void for_steps(F f) {
    const StepTable<PT, NP, UT> t;
    for (int i = 0; i < t.n; ++i) f(t.ph[i] / NP, t.ph[i] % NP, t.oy[i], t.xs[i], t.rem[i], t.late[i]);
}

template <class F>
void pat_steps(int pat, int ut, F f) {
#define MNB_PS(P_, NP_)                              \
    if (ut == 1) for_steps<P_, NP_, 1>(f);           \
    else if (ut == 2) for_steps<P_, NP_, 2>(f);      \
    else for_steps<P_, NP_, 4>(f);                   \
    break;
    switch (pat) {
        case PAT_F31: MNB_PS(P3, 1)
        case PAT_F21: MNB_PS(P2, 1)
        case PAT_F42: MNB_PS(P4, 1)
        case PAT_F32: MNB_PS(P3, 1)
        case PAT_F12: MNB_PS(P1, 1)
        case PAT_T42D: MNB_PS(P42D, 2)
        case PAT_T42S: MNB_PS(P42S, 2)
        case PAT_T32D: MNB_PS(P32D, 2)
        case PAT_T32S: MNB_PS(P32S, 2)
        default: MNB_PS(P1, 2)
    }
#undef MNB_PS
}

int pat_nd(int pat) {
    switch (pat) {
        case PAT_F31: case PAT_F32: case PAT_T42D: return 3;
        case PAT_F42: return 4;
        case PAT_F12: case PAT_T12: return 1;
        default: return 2;
    }
}
int pat_s(int pat) { return pat == PAT_F42 || pat == PAT_F32 || pat == PAT_F12 ? 2 : 1; }
int pat_np(int pat) { return pat >= PAT_T42D ? 2 : 1; }

// Stride-2 forward filters stage one 8-channel group at a time: their windows are four times their
// tiles, and with more groups a workgroup's LDS leaves one or two of them on a compute unit (32x32x32
// -> 16x16x32 4x4 / 2: 140 TFLOP/s with one group, 109 with two, 85 with four; 16x16x16 -> 8x8x32
// 3x3 / 2: 98 / 68).  The others gain from fewer stages (32x16x16 -> 64 3x3 / 1: 173 / 174 / 211).
bool one_group(int pat) { return pat == PAT_F42 || pat == PAT_F32; }

// The convolution as the kernel sees it.
struct View {
    int Cin, Cout, Hi, Wi, Ho, Wo, oH, oW;
};
View view_of(const ConvGeom& g, bool back, int pat) {
    View v;
    v.Cin = back ? g.Co : g.Ci; v.Cout = back ? g.Ci : g.Co;
    v.Hi = back ? g.Ho : g.Hi; v.Wi = back ? g.Wo : g.Wi;
    v.oH = back ? g.Hi : g.Ho; v.oW = back ? g.Wi : g.Wo;
    const int np = pat_np(pat);
    v.Ho = (v.oH + np - 1) / np; v.Wo = (v.oW + np - 1) / np;
    return v;
}

struct Tile {
    int FN, FM, WN, WM;
    int BM() const { return 16 * FM * WM; }
    int BN() const { return 16 * FN * WN; }
};

// Launch shape of one tile: rows per workgroup, tiles per row, window, LDS.
struct Shape {
    int R, mtiles, WH, RS, plane;
    size_t lds;
    double fill;   // share of the tile's positions that exist
};
Shape shape_of(const View& v, int pat, int pad, int cgs, const Tile& t) {
    Shape s;
    const int P = v.Ho * v.Wo, S = pat_s(pat), nd = pat_nd(pat), BM = t.BM();
    s.RS = std::max(S * (v.Wo - 1) + nd, pad + v.Wi);
    // positions per channel group, 1 mod 16: the groups that the lanes of a fragment read then start 48
    // bytes apart modulo the banks, like its neighbouring positions (at 64 bytes, 108 positions, 43% of the
    // LDS cycles were conflicts)
    auto planes = [&](int rows) { return cgs == 1 ? rows * s.WH * s.RS : (rows * s.WH * s.RS + 14) / 16 * 16 + 1; };
    auto lds = [&](int rows) { return ((size_t)cgs * planes(rows) + 1) * POSB; };
    if (P <= BM) {
        s.mtiles = 1;
        s.WH = S * (v.Ho - 1) + nd;
        s.R = BM / P;
        while (s.R > 1 && lds(s.R) > SPLIT_LDS_ROWS) --s.R;
        s.fill = (double)s.R * P / BM;
    } else {
        s.R = 1;
        s.mtiles = cdiv(P, BM);
        s.WH = 0;
        for (int mt = 0; mt < s.mtiles; ++mt) {
            const int yf = mt * BM / v.Wo, yl = (std::min((mt + 1) * BM, P) - 1) / v.Wo;
            s.WH = std::max(s.WH, S * (yl - yf) + nd);
        }
        s.fill = (double)P / ((double)s.mtiles * BM);
    }
    s.plane = planes(s.R);
    s.lds = lds(s.R);
    return s;
}

// Tiles that serve Cout channels, the preferred one first (launch_split leaves it where another one's
// positions are better filled).
int tiles_for(int pat, int Cout, Tile* t) {
    int n = 0;
    if (pat_np(pat) == 1) {
        if (Cout % 64 == 0) { t[n++] = Tile{2, 4, 2, 2}; t[n++] = Tile{2, 2, 2, 2}; }
        else if (Cout % 32 == 0) { t[n++] = Tile{2, 2, 1, 4}; t[n++] = Tile{2, 4, 1, 4}; t[n++] = Tile{2, 1, 1, 4}; }
        else { t[n++] = Tile{1, 2, 1, 4}; t[n++] = Tile{1, 4, 1, 4}; }
    } else {
        // (two position fragments a wavefront: with four, the four phases' accumulators leave no registers)
        t[n++] = Cout % 64 == 0 ? Tile{1, 2, 4, 1} : Cout % 32 == 0 ? Tile{1, 2, 2, 2} : Tile{1, 2, 1, 4};
    }
    return n;
}

template <class PT, int NP, int S>
void launch_pat(const Tile& t, int cgs, dim3 grid, size_t lds, const SplitArgs& a, hipStream_t st) {
#define MNB_SP(C_, FN_, FM_, WN_, WM_)                                                              \
    if (cgs == C_ && t.FN == FN_ && t.FM == FM_ && t.WN == WN_ && t.WM == WM_) {                    \
        hipLaunchKernelGGL((k_conv_split<PT, NP, S, C_, FN_, FM_, WN_, WM_>), grid, dim3(64 * WN_ * WM_), lds, st, a); \
        MNB_HIP(hipGetLastError());                                                                 \
        return;                                                                                     \
    }
#define MNB_SPC(FN_, FM_, WN_, WM_)                                                                 \
    MNB_SP(1, FN_, FM_, WN_, WM_)                                                                   \
    if constexpr (!(S == 2 && PT::cnt(0) > 1)) { MNB_SP(4, FN_, FM_, WN_, WM_) MNB_SP(2, FN_, FM_, WN_, WM_) }
    if constexpr (NP == 1) {
        MNB_SPC(2, 4, 2, 2) MNB_SPC(2, 2, 2, 2)
        MNB_SPC(2, 2, 1, 4) MNB_SPC(2, 4, 1, 4) MNB_SPC(2, 1, 1, 4)
        MNB_SPC(1, 2, 1, 4) MNB_SPC(1, 4, 1, 4)
    } else {
        MNB_SPC(1, 2, 4, 1) MNB_SPC(1, 2, 2, 2) MNB_SPC(1, 2, 1, 4)
    }
#undef MNB_SPC
#undef MNB_SP
    throw Error{MNB_EDEVICE, "no such convolution tile"};
}

bool launch_split(const ConvGeom& g, const SplitConv& sc, bool back, const float* in, float* out, int M, bool accumulate,
                  hipStream_t st, const ConeClip* clip) {
    if (sc.w == nullptr) return false;
    const View v = view_of(g, back, sc.pat);
    Tile ts[4];
    const int nt = tiles_for(sc.pat, v.Cout, ts);
    int best = -1;
    double score = 0;
    Shape sh{};
    for (int i = 0; i < nt; ++i) {
        const Shape s = shape_of(v, sc.pat, sc.pad, sc.cgs, ts[i]);
        if (s.lds > SPLIT_LDS_MAX) continue;
        // (4x4 / 2 into 32 channels on whole 256-position grids: four fragments a wavefront, 139 against 128
        // TFLOP/s at 32x32x32)
        const bool wide = sc.pat == PAT_F42 && ts[i].WN == 1 && ts[i].FM == 4 && v.Ho * v.Wo >= 256;
        const double q = s.fill * (wide ? 1.05 : i == 0 ? 1.0 : 0.8);
        if (q > score) { score = q; best = i; sh = s; }
    }
    if (best < 0) return false;
    const Tile& t = ts[best];
    SplitArgs a{};
    a.G = in; a.C = out; a.Ws = sc.w; a.bias = back ? nullptr : g.b;
    a.ldG = (long)v.Cin * v.Hi * v.Wi; a.ldC = (long)v.Cout * v.oH * v.oW;
    a.M = M; a.Hi = v.Hi; a.Wi = v.Wi; a.Co = v.Cout; a.Ho = v.Ho; a.Wo = v.Wo; a.p = sc.pad;
    a.R = sh.R; a.mtiles = sh.mtiles; a.P = v.Ho * v.Wo; a.ng = cdiv(v.Cin, 8 * sc.cgs); a.acc = accumulate;
    a.WH = sh.WH; a.RS = sh.RS; a.plane = sh.plane;
    a.oH = v.oH; a.oW = v.oW;
    a.clip = clip ? *clip : ConeClip{};
    a.rWo = 1.f / (float)v.Wo; a.rP = 1.f / (float)a.P; a.rWi = 1.f / (float)v.Wi;
    const bool al = ((uintptr_t)out & 15) == 0 && a.ldC % 4 == 0 && (v.oH * v.oW) % 4 == 0;
    a.quad = pat_np(sc.pat) == 1 ? al && a.P % 4 == 0 : ((uintptr_t)out & 7) == 0 && v.oW % 2 == 0;
    const long gx = sh.R > 1 ? cdiv(M, sh.R) : (long)M * sh.mtiles;
    if (gx > 0x7fffffffL) return false;
    const dim3 grid((unsigned)gx, v.Cout / t.BN());
    switch (sc.pat) {
        case PAT_F21: launch_pat<P2, 1, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_F31: launch_pat<P3, 1, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_F42: launch_pat<P4, 1, 2>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_F32: launch_pat<P3, 1, 2>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_F12: launch_pat<P1, 1, 2>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_T42D: launch_pat<P42D, 2, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_T42S: launch_pat<P42S, 2, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_T32D: launch_pat<P32D, 2, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        case PAT_T32S: launch_pat<P32S, 2, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
        default: launch_pat<P1, 2, 1>(t, sc.cgs, grid, sh.lds, a, st); break;
    }
    return true;
}

// Pattern, padding and channel groups per stage of one direction of a convolution; sc.cgs = 0: not
// covered.
void plan_split(const ConvGeom& g, bool back, SplitConv& sc) {
    sc = SplitConv{};
    const int k = g.k, s = g.s;
    if (!back) {
        if (g.p < 0) return;
        if (k == 3 && s == 1) sc.pat = PAT_F31;
        else if (k == 2 && s == 1) sc.pat = PAT_F21;
        else if (k == 4 && s == 2) sc.pat = PAT_F42;
        else if (k == 3 && s == 2) sc.pat = PAT_F32;
        else if (k == 1 && s == 2) sc.pat = PAT_F12;
        else return;
        sc.pad = g.p;
    } else if (s == 1) {
        if ((k != 3 && k != 2) || g.p > k - 1) return;
        sc.pat = k == 3 ? PAT_F31 : PAT_F21;
        sc.pad = k - 1 - g.p;
    } else {
        if (s != 2 || g.n_phase != 4 || g.Hi < 2 || g.Wi < 2) return;
        // phases by output parity: pads and taps per dimension (rows and columns alike)
        int O[2] = {0, 0}, N[2] = {0, 0}, pad[2] = {0, 0};
        for (int f = 0; f < 4; ++f) {
            const ConvPhase& ph = g.ph[f];
            if (ph.rho_y != ph.rho_x) continue;
            N[ph.Y0] = ph.Ty;
            pad[ph.Y0] = ph.Ty - 1 - ph.q0y;
        }
        int pm = -1000;
        for (int a = 0; a < 2; ++a)
            if (N[a] > 0) pm = std::max(pm, pad[a]);
        for (int a = 0; a < 2; ++a)
            if (N[a] > 0) O[a] = pm - pad[a];
        auto is = [&](int o0, int n0, int o1, int n1) { return O[0] == o0 && N[0] == n0 && O[1] == o1 && N[1] == n1; };
        if (is(0, 2, 1, 2)) sc.pat = PAT_T42D;
        else if (is(0, 2, 0, 2)) sc.pat = PAT_T42S;
        else if (is(0, 1, 0, 2)) sc.pat = PAT_T32D;
        else if (is(0, 2, 1, 1)) sc.pat = PAT_T32S;
        else if (is(0, 1, 0, 0)) sc.pat = PAT_T12;
        else return;
        if (pm < 0) return;
        sc.pad = pm;
    }
    const View v = view_of(g, back, sc.pat);
    if (v.Cin % 8 != 0 || v.Cout % 16 != 0 || v.Ho < 1 || v.Wo < 1) return;
    Tile ts[4];
    tiles_for(sc.pat, v.Cout, ts);
    for (int c : {4, 2, 1}) {
        if (v.Cin % (8 * c) != 0 || (c > 1 && one_group(sc.pat))) continue;
        if (shape_of(v, sc.pat, sc.pad, c, ts[0]).lds <= SPLIT_LDS_MAX) {
            sc.cgs = c;
            break;
        }
    }
}

}  // namespace

size_t split_stream_bytes(ConvGeom& g, bool back) {
    SplitConv& sc = back ? g.sb : g.sf;
    plan_split(g, back, sc);
    if (sc.cgs == 0) return 0;
    const View v = view_of(g, back, sc.pat);
    int nstep = 0;
    pat_steps(sc.pat, 4 / sc.cgs, [&](int, int, int, int, int, bool) { ++nstep; });
    sc.nstep = nstep;
    // one more step: the kernel fetches a step ahead
    return ((size_t)(v.Cout / 16) * (v.Cin / (8 * sc.cgs)) * nstep + 1) * STEPB;
}

void launch_split_stream(ConvGeom& g, bool back, void* out, hipStream_t st) {
    SplitConv& sc = back ? g.sb : g.sf;
    const View v = view_of(g, back, sc.pat);
    const int ut = 4 / sc.cgs;
    StreamArgs a{};
    a.W = g.W; a.out = (unsigned short*)out;
    a.Cin = v.Cin; a.Cout = v.Cout; a.k = g.k; a.back = back; a.ng = v.Cin / (8 * sc.cgs); a.cgs = sc.cgs;
    a.nstep = sc.nstep;
    int t = 0;
    pat_steps(sc.pat, ut, [&](int pa, int pb, int oy, int xs, int rem, bool late) {
        for (int u = 0; u < ut; ++u) {
            int ky = oy, kx = xs + u;
            if (back) {
                // phase a reads coefficient y + o - pad through tap ty = q0 + pad - o, filter row rho + s ty
                auto tap = [&](int a_, int o, bool row) {
                    for (int f = 0; f < g.n_phase; ++f) {
                        const ConvPhase& ph = g.ph[f];
                        if ((row ? ph.Y0 : ph.X0) != a_) continue;
                        return row ? ph.rho_y + g.s * (ph.q0y + sc.pad - o) : ph.rho_x + g.s * (ph.q0x + sc.pad - o);
                    }
                    return -1;
                };
                ky = tap(pa, oy, true);
                kx = tap(pb, xs + u, false);
            }
            a.tap[t * ut + u] = u < rem ? (short)(ky << 8 | kx) : (short)-1;
        }
        if (late) a.late |= 1ull << t;
        ++t;
    });
    const long n = (long)(v.Cout / 16) * a.ng * sc.nstep * 512;
    hipLaunchKernelGGL(k_split_stream, dim3(cdiv(n, 256)), dim3(256), 0, st, a, n);
    MNB_HIP(hipGetLastError());
    sc.w = (const unsigned char*)out;
}

bool launch_conv_forward_split(const ConvGeom& g, const float* G, float* C, int M, bool accumulate, hipStream_t st,
                               const ConeClip* clip) {
    if (kernel_variants() & MNB_VAR_NO_WIN_CONV) return false;
    return launch_split(g, g.sf, false, G, C, M, accumulate, st, clip);
}
bool launch_conv_backsub_split(const ConvGeom& g, const float* A, float* C, int M, bool accumulate, hipStream_t st) {
    if (kernel_variants() & MNB_VAR_NO_WIN_CONV) return false;
    return launch_split(g, g.sb, true, A, C, M, accumulate, st, nullptr);
}

}  // namespace mnb
