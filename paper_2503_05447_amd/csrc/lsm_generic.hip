// Generic kernel family of the chunkwise LSM path: fp32 arithmetic for any supported (d_k, d_v, chunk) and both
// element types.  It is the product path for fp32 inputs (whose 1e-4 tolerance rules out bf16 operands) and for the
// shapes the bf16 family does not cover (64-wide heads, chunk sizes other than 64).
//
// Everything is one walker, gk_walk.  With roles query x, key y, value z and a running state
//     out_p = e^{E_p} x_p S + sum_{s <= p} (x_p . y_s) e^{E_p - E_s} z_s ,   S <- e^{E} S + sum_s e^{E - E_s} y_s^T z_s
// (p: position in walk order, E: running log-decay), the forward pass and all three gradients are the same product with
// the operands in different roles (the adjoint walks backward in time):
//     o : (q, k, v) forward      dq : (d_o, v, k) forward      dv : (k, q, d_o) backward      dk : (v, d_o, q) backward
// so no per-chunk state or state gradient ever reaches memory: a workgroup walks a segment of a sequence 32 tokens at a
// time with its state in matrix-core accumulators.  Where a launch has too few sequences a sequence is cut into
// segments: gk_walk<SUM> (state update alone, from zero) leaves every segment's own contribution, gk_scan chains them,
// and the walkers then run all segments in parallel.  The decay gradient needs, per token, q.dq and k.dk (left by the
// two walkers) and, per chunk, the product of the state and its gradient at the chunk's end: the dq walker leaves its state
// there, the dk walker, launched after it, multiplies it with its own, and gk_dg sums backward from there.  (Summing back
// from the end of a whole segment needs no state per chunk, but the roundings of q.dq and k.dk add up over the way: 2-norm
// error 2.2e-6 against 3.6e-7 with segments of 2048 tokens and a decay of e^-0.02 a token.)
//
// Contractions of the vector kind are v_mfma_f32_32x32x2_f32 (but where bf16 rows enter as they came, see gk_walk_vec): fp32 operands, fp32 accumulation, 1/16 of the bf16 rate but exact
// products, and its operand layout is its result layout: lane l holds A[m = l%32][k = l/32], B[k = l/32][n = l%32], and result
// register 4g+j of lane l is D[m = 8g + 4(l/32) + j][n = l%32].  Register x of a result block is therefore, unchanged, the
// operand of one MFMA of the next product (its k index are the rows 8g+j and 8g+4+j), so states and scores feed the
// matrix cores straight out of the accumulators and nothing is split or rounded on the way.  The scalar kinds run the same
// products on the bf16 matrix cores, operands in three parts (below).
//
// Bound: the vector ALU and its order with the matrix instructions.  Scalar kinds, 4 x 16 sequences of 2047 fp32 tokens, d = 128:
// vector issue 55 %, matrix pipes 30 % of the walk (fp32 instructions alone: matrix pipes 54 %, the whole step 18 % longer); the
// vector kind its chain of phases: 26000 to 28000 clocks a step, of which each of the two groups works some 20000.
// Forward + backward against one-thread-per-element kernels on the vector ALU with a state per chunk in memory, which this
// family replaced, then with fp32 instructions throughout, now: that shape 11.6 ms, 0.731, 0.621; bf16 vector decay, 4 x 8
// sequences of 2048, d_k = 64, d_v = 128: 7.2 ms, 0.442, 0.357; forward alone, 32 sequences of 1777, d = 64, bf16: 262 us, 50.7,
// 43.5; 2 sequences of 256, d = 64, fp32: 110 us, 25.1, 23.6.
// Distance to 64-bit results against the kernels on the vector ALU, 2-norm, weak to strong decays, 512 to 4096 tokens, chunks of 16
// to 128: o, dq, dk, dv and d_init_state 0.4 to 0.95 times (one case 1.09), dg 0.1 to 0.85 times (vector kind in chunks of 16: 1.04),
// the final state 0.7 to 1.2 times (at most 5.5e-8 where it was 5.0e-8); the scalar kinds in three parts are closer again (fp32, 2
// sequences of 256, d = 64: 1.6e-7 -> 8.8e-8; training step at 4 x 16 x 2047: furthest output 4.2e-7 -> 4.0e-7).
#include "lsm_internal.h"

#include <algorithm>
#include <cfloat>
#include <initializer_list>
#include <mutex>
#include <vector>

namespace lsm {
namespace {

constexpr int GT = 32;  // tokens per step of a walk
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ uint32_t bf16_bits(float x) {  // round to nearest even, NaN kept quiet
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
// four consecutive elements
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const uint16_t* p) {
    const u32x2 w = *reinterpret_cast<const u32x2*>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
}
// the same in two steps: as they lie in memory, then as numbers
__device__ __forceinline__ f32x4 load4raw(const float* p) { return load4(p); }
__device__ __forceinline__ u32x2 load4raw(const uint16_t* p) { return *reinterpret_cast<const u32x2*>(p); }
__device__ __forceinline__ f32x4 numbers4(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 numbers4(u32x2 w) {
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store4(uint16_t* p, f32x4 v) {
    *reinterpret_cast<u32x2*>(p) = u32x2{bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16)};
}

// One operand assignment of the walk.
struct GRole {
    const void *xq, *xk, *xv;  // rows in the query, key and value role
    const void* aux;           // rows the unrounded output is multiplied with for the decay gradient, or NULL
    void* out;
    float* xdot;               // that product: scalar kinds [value slice][BH*T] (summed over the row), vector kind [BH*T][width]
    const float* edge_in;      // state the whole sequence starts from (walk order), [d_k][d_v] per sequence; NULL = zero
    float* edge_out;           // state it ends with; NULL = not wanted
    float* bound;              // states at segment boundaries, [d_k][d_v] each (bound_at)
    double* gseg;              // SUM: total log-decay of each segment ([slot], vector kind [slot][d_k])
    int rev, trans;            // walk backward in time; the walk's state is the transpose of the stored one
    int per;                   // 0: bound is numbered by segments; else by decay-gradient units, so many to a segment
    int keep;                  // leave the state at the end of every unit in bound (1: but not the sequence's last, 2: all)
    const float* dot;          // such states of the other direction: their products with this walk's state go to z,
    double* z;                 //   [unit][width / 32] (one term per wave), vector kind [unit][2][width] (one per group)
};
struct GArgs {
    GRole role[3];
    const float* g;
    int kd, vd;        // row widths of the key-role and value-role arrays
    int nsl;           // value slices (grid.z = role * nsl + slice)
    int m;             // segment length in units of Dims::gC tokens
    int slots;         // boundary slots per head (packed input) or per sequence
    int units;         // units of Dims::gC tokens per head (packed input) or per sequence
};

// Unit of the decay gradient: the tokens its sums run back over.
__host__ __device__ __forceinline__ int dg_unit(const Dims& d) { return d.C < GT ? GT : d.C; }
__host__ __device__ __forceinline__ int dg_per(const Dims& d) { return d.gC / dg_unit(d); }  // such units per unit of gC tokens

// Segment `x` of the grid: packed input numbers the segments of all sequences of a head one after the other, sequence s
// from its first unit / m + s on (units counted per sequence and at least one each, so that two never overlap).
struct GSeg { SeqWalk w; int n, seg, nsq; size_t slot0, unit0; };
__device__ __forceinline__ int seg_base(const Dims& d, int m, int s) { return m == 1 ? d.cstart[s] : d.cstart[s] / m + s; }
// last sequence s with base(s) <= x (base ascending), 64 sequences at a time, one per lane
template <typename F>
__device__ __forceinline__ int last_seq(const Dims& d, int x, F base) {
    int lo = -1;
    for (int s0 = 0; s0 < d.nseq; s0 += 64) {
        const int t = s0 + int(threadIdx.x & 63);
        const uint64_t le = __ballot(t < d.nseq && base(min(t, d.nseq)) <= x);
        lo += __popcll(le);
        if (le != ~uint64_t(0)) break;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}
__device__ __forceinline__ GSeg find_seg(const Dims& d, const GArgs& a, int x, int y) {
    GSeg r;
    if (!d.cu) {
        r.w = SeqWalk{y, y, 0, 0, 0, d.T};
        r.seg = x;
        r.slot0 = size_t(y) * a.slots;
        r.unit0 = size_t(y) * a.units;
    } else {
        const int lo = last_seq(d, x, [&](int s) { return seg_base(d, a.m, s); });
        r.w = SeqWalk{y, lo * d.H + y, 0, 0, d.cu[lo], d.cu[lo + 1]};
        r.seg = x - seg_base(d, a.m, lo);
        r.slot0 = size_t(y) * a.slots + seg_base(d, a.m, lo);
        r.unit0 = size_t(y) * a.units + d.cstart[lo];
    }
    r.unit0 *= dg_per(d);
    const int len = r.w.tend - r.w.tbeg;
    r.n = (len + GT - 1) / GT;
    r.nsq = (len + d.gC * a.m - 1) / (d.gC * a.m);
    return r;
}
// slot of the state that segment w >= 1 (walk order) starts from: the one at the end of the unit before it
__device__ __forceinline__ size_t bound_at(int per, size_t slot0, size_t unit0, int w) {
    return per ? unit0 + size_t(w) * per - 1 : slot0 + w;
}

// one operand's 32 rows on their way to LDS: 16-byte pieces, dealt to the threads row by row
template <typename TIO, int W, int NT>
struct GTile {
    static constexpr int PER = 16 / int(sizeof(TIO)), PR = W / PER, CNT = GT * PR / NT;
    static_assert(CNT * NT == GT * PR, "tile pieces divide evenly");
    u32x4 v[CNT];
    // uniform base + a 32-bit byte offset per lane; rows beyond the ragged end repeat the last one and are zeroed later
    __device__ __forceinline__ void gload(const TIO* base, uint32_t rowbytes, int L, int rev, int tid) {
        const char* b = reinterpret_cast<const char*>(base);
        _Pragma("unroll") for (int i = 0; i < CNT; ++i) {
            const int p = tid + NT * i, row = min(p / PR, L - 1), c = p % PR;
            v[i] = *reinterpret_cast<const u32x4*>(b + (uint32_t(rev ? L - 1 - row : row) * rowbytes + uint32_t(c * 16)));
        }
    }
    __device__ __forceinline__ void clear(int L, int tid) {  // rows beyond the ragged end
        if (L < GT)
            _Pragma("unroll") for (int i = 0; i < CNT; ++i)
                if ((tid + NT * i) / PR >= L) v[i] = u32x4{0, 0, 0, 0};
    }
    __device__ __forceinline__ void commit(float* dst, int ld, int L, int tid) const {
        _Pragma("unroll") for (int i = 0; i < CNT; ++i) {
            const int p = tid + NT * i, row = p / PR, c = p % PR;
            const uint32_t keep = row < L ? 0xffffffffu : 0u;
            const u32x4 x = {v[i].x & keep, v[i].y & keep, v[i].z & keep, v[i].w & keep};
            float* q = dst + row * ld + c * PER;
            if (PER == 4) {
                *reinterpret_cast<u32x4*>(q) = x;
            } else {
                *reinterpret_cast<u32x4*>(q) = u32x4{x.x << 16, x.x & 0xffff0000u, x.y << 16, x.y & 0xffff0000u};
                *reinterpret_cast<u32x4*>(q + 4) = u32x4{x.z << 16, x.z & 0xffff0000u, x.w << 16, x.w & 0xffff0000u};
            }
        }
    }
};

// state blocks <-> a stored state [d_k][d_v] (rows are key features; trans: value features): S[ib][4g+j] = state[key feature
// kf + 32 ib + 8g + 4 half + j][value feature vf + lane % 32]
template <int KB>
__device__ __forceinline__ void state_load(f32x16 (&S)[KB], const float* e, int trans, int kd, int vd, int kf, int vf, int lane) {
    const int v = vf + (lane & 31);
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            const int k = kf + 32 * ib + 8 * g + 4 * (lane >> 5);
            if (trans) {
                const f32x4 t = load4(e + size_t(v) * kd + k);
                _Pragma("unroll") for (int j = 0; j < 4; ++j) S[ib][4 * g + j] = t[j];
            } else {
                _Pragma("unroll") for (int j = 0; j < 4; ++j) S[ib][4 * g + j] = e[size_t(k + j) * vd + v];
            }
        }
}
template <int KB>
__device__ __forceinline__ void state_store(const f32x16 (&S)[KB], float* e, int trans, int kd, int vd, int kf, int vf, int lane) {
    const int v = vf + (lane & 31);
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            const int k = kf + 32 * ib + 8 * g + 4 * (lane >> 5);
            if (trans) {
                store4(e + size_t(v) * kd + k, f32x4{S[ib][4 * g], S[ib][4 * g + 1], S[ib][4 * g + 2], S[ib][4 * g + 3]});
            } else {
                _Pragma("unroll") for (int j = 0; j < 4; ++j) e[size_t(k + j) * vd + v] = S[ib][4 * g + j];
            }
        }
}
// this lane's part of the product of two states: S and the stored one, transposed (elements as in state_load with trans)
template <int KB>
__device__ __forceinline__ double state_dot(const f32x16 (&S)[KB], const float* e, int kd, int kf, int vf, int lane) {
    double z = 0.0;
    e += size_t(vf + (lane & 31)) * kd + kf + 4 * (lane >> 5);
    f32x4 t[KB][4];  // every load before the first use (64 KiB of states: four trips to memory instead of one took 7500 clocks)
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
        _Pragma("unroll") for (int g = 0; g < 4; ++g) t[ib][g] = load4(e + 32 * ib + 8 * g);
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
        _Pragma("unroll") for (int x = 0; x < 16; ++x) z += double(t[ib][x >> 2][x & 3]) * double(S[ib][x]);
    return z;
}
__device__ __forceinline__ int hrow(int x, int half) { return 8 * (x >> 2) + 4 * half + (x & 3); }  // row of result register x

// X[v][p] = sum_s Z[s][v] P[s][p]: the score block as B operand out of its registers, `z` at value feature 0 of this wave.
// P is zero where s does not precede p, but a zero times an infinity or NaN is not: a value row that is not finite would
// reach the positions before it, which must not depend on it.  Where the block holds one (seen on the operands as they are
// loaded) the matrix product runs without such elements and they are added pair by pair, ok(s, p) only.  The check costs nothing:
// forward + backward, bf16 vector decay, 4 x 8 sequences of 2048, d_k = 64, without and with it 444 / 442 us.
// LV: a level's block (0: any): rows on its odd side are zero, and where that can be told from the register alone they are left out.
template <int LV, typename Ok>
__device__ __forceinline__ f32x16 causal_product(const float* z, int ld, const f32x16& P, int lane, Ok ok) {
    const int n = lane & 31, half = lane >> 5;
    constexpr int skip = LV == 4 ? 0 : LV;  // (register x: row 8 (x / 4) + 4 half + x % 4)
    f32x16 X = {0};
    float chk = 0.f;
    _Pragma("unroll") for (int x = 0; x < 16; ++x) {
        if (hrow(x, 0) & skip) continue;
        const float t = z[hrow(x, half) * ld + n];
        chk = fmaf(t, 0.f, chk);
        X = mfma2(t, P[x], X);
    }
    if (__any(chk != chk)) {
        X = f32x16{0};
        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
            if (hrow(x, 0) & skip) continue;
            const float t = z[hrow(x, half) * ld + n];
            X = mfma2(fabsf(t) <= FLT_MAX ? t : 0.f, P[x], X);
        }
        _Pragma("unroll 1") for (int s = 0; s < GT; ++s) {
            const float p = __shfl(P[4 * (s >> 3) + (s & 3)], n + 8 * (s & 4), 64);  // P[s][n]
            _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                const f32x4 t = *reinterpret_cast<const f32x4*>(z + s * ld + 8 * g + 4 * half);
                _Pragma("unroll") for (int j = 0; j < 4; ++j)
                    if (ok(s, n) && !(fabsf(t[j]) <= FLT_MAX)) X[4 * g + j] += t[j] * p;
            }
        }
    }
    return X;
}

// Have a block in its registers here.  Left alone the compiler puts what is added to a block in every phase off until the block is
// used, phases later, and keeps the operands instead: gk_walk_vec's outputs, five levels of them, went through scratch memory,
// behind every store before (20000 of 43000 clocks a step, bf16, d_k = 64, d_v = 128).  (o and dv of 64-wide values: with 256 decayed
// features 2 to 4 % shorter with it, fp32, 4 x 8 sequences of 2048 forward 507 and 486 us; with fewer up to 2 % longer, not there.)
__device__ __forceinline__ void formed(f32x16& x) { asm volatile("" : "+v"(x)); }

// What a workgroup walks.
struct GWalk {
    SeqWalk walk;
    size_t slot0, unit0;
    int n, nsq, kbeg, kend, cnt, wseg;  // steps and segments of the sequence; steps [kbeg, kend); segment index in walk order
    bool empty;                      // packed input, an empty sequence: the state passes through
    bool none;                       // no work
    ChunkPos origin;                 // of the head's token 0
};
__device__ __forceinline__ GWalk find_walk(const Dims& d, const GArgs& a, int rev, bool sum) {
    const GSeg s = find_seg(d, a, blockIdx.x, blockIdx.y);
    const int steps = a.m * (d.gC / GT), kbeg = s.seg * steps, kend = min(s.n, kbeg + steps);
    GWalk g{s.w, s.slot0, s.unit0, s.n, s.nsq, kbeg, kend, max(kend - kbeg, 0), rev ? s.nsq - 1 - s.seg : s.seg, s.n == 0 && s.seg == 0, false, chunk_pos_at(d, s.w.bh, 0, 0, 0)};
    g.none = (s.seg >= s.nsq && !g.empty) || (sum && g.wseg >= s.nsq - 1);  // (nobody starts from the last segment's end)
    return g;
}
// position of the kk-th step; past the last it is one row of it, that nobody uses: rows are requested a step ahead and
// unconditionally (behind a branch the old values would stay live through the whole step)
__device__ __forceinline__ ChunkPos walk_step(const Dims& d, const GWalk& g, int rev, int kk) {
    const int k = min(kk, g.cnt - 1), t0 = g.walk.tbeg + (rev ? g.kend - 1 - k : g.kbeg + k) * GT;
    ChunkPos p = g.origin;  // (head and batch are told apart once: a division per step is a chain of a hundred clocks)
    p.t0 = t0;
    p.L = kk >= g.cnt ? 1 : min(GT, g.walk.tend - t0);
    p.tok0 += size_t(t0) * p.ts;
    p.wtok0 += t0;
    return p;
}

// decay-gradient unit that ends with the kk-th step, -1 if none does
__device__ __forceinline__ int unit_end(const Dims& d, const GWalk& g, int rev, int kk) {
    const int k = rev ? g.kend - 1 - kk : g.kbeg + kk, steps = dg_unit(d) / GT;
    return (k + 1) % steps == 0 || k + 1 == g.n ? k / steps : -1;
}
// slot for the state after the kk-th step of a walk that keeps the units' states, -1 if that is not kept: at the end of a
// segment the slot has the next segment's entry state already
__device__ __forceinline__ long long keep_slot(const Dims& d, const GRole& R, const GWalk& g, int kk) {
    if (!R.keep || (kk == g.cnt - 1 && (g.wseg < g.nsq - 1 || R.keep < 2))) return -1;
    const int u = unit_end(d, g, R.rev, kk);
    return u < 0 ? -1 : (long long)(g.unit0 + u);
}

// LDS of the vector kind's walker, in floats.  Row strides == 4 mod 64 words: 16-byte row reads of 16 lanes tile the banks.
//   Q | K | V | score partials, then half of the inter product [wave][16][64] | W (one or two tiles of weighted rows) | tables
// bf16 elements: the rows that enter products as they came stay bf16 (GRows), keys and queries of VEC 2, values of
// the summary (64-wide ones not: forward, 8 sequences of 2000, d = 64, 43.5 -> 46 us).
template <typename TIO, int KD, int TV, int VEC, bool SUM>
struct GLds {
    static constexpr bool RAW = sizeof(TIO) == 2 && (VEC == 2 || (SUM && TV == 128));
    static constexpr int NW = TV / 32, LQ = KD + 4, LV = TV + 4;
    static constexpr int COLS = VEC == 2 ? TV : KD;           // decayed features held by this workgroup
    static constexpr int QK = RAW && VEC == 2 ? GT * (KD + 8) / 2 : GT * LQ, VT = RAW && VEC == 1 ? GT * (TV + 8) / 2 : GT * LV;
    static constexpr int WT = GT * (COLS + 4), WN = SUM ? 1 : 2;
    static constexpr int oK = SUM ? 0 : QK, oV = oK + QK, oP = oV + VT, oW = oP + (SUM ? 0 : NW * 1024);
    // a decayed feature's 32 positions are dealt to 2 threads of the group that weighs rows, or to 4 where there are as many (of the
    // supported shapes d_k = 64, d_v = 128 alone: o and dv, and the summary): then the sums of four pieces, and their products for the
    // level whose blocks are two pieces (4 x 8 sequences of 2048, with 2: o and dv walkers 77 us, summary 37; with 4: 71 and 33)
    static constexpr int PIECES = 4 * COLS <= 2 * TV ? 4 : 2;
    static constexpr int oT = oW + WN * WT, total = oT + (PIECES == 4 ? 17 : 5) * COLS, bytes = total * 4;
};

// ---- fp32 products on the bf16 matrix cores
//
// An fp32 number of 2^-110 and more is the sum of three bf16 ones exactly (head = rounded, then the rounded remainder, then what
// is left), so a product of two of them is a handful of bf16 products accumulated in fp32: six where both operands are split
// (the three of 2^-25 and less are dropped), three where one of them is a bf16 number to begin with.  At 16 times the rate of
// the fp32 matrix instructions that is 3/8 or 3/16 of their time, and closer: 16 terms are added per rounding instead of 2, and
// the small products, added apart or first, are not rounded at the size of the sum.  One 32 x 32 block of normal numbers,
// K = 128, 2-norm error against 64 bits: fp32 instructions 2.0e-7, six products 8.8e-8, three 6.4e-8.
//
// Below that the last parts, or their low bits, would be under the smallest bf16 number.  So what is split is 2^24 times the
// operand, which gives every normal number three parts that are normal, and the result's factor is taken out of the sum: the
// same bits, over the whole range of fp32.  Cost, forward + backward, fp32, 4 x 16 sequences of 2047, d = 128: 605 -> 621 us;
// forward, bf16, 32 sequences of 1777, d = 64: 42.2 -> 43.5; at most 7 % (forward + backward, bf16, 32 of 1777, d_k = 64, d_v = 128:
// 191 -> 205; with fp32 instructions throughout 296).
//
// What is not finite has no such sum (infinity - infinity), and 2^24 times a number of 2^104 and more is not finite: elements of a result
// that are not finite are formed again with the fp32 instructions from the numbers themselves (rows and states from where they
// came from, a score from its parts, which then hold its bits).  The others stay as they are, so that they do not depend on
// what is not finite.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2)); }
__device__ __forceinline__ float lo2(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi2(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
constexpr float kUp = 0x1p24f, kDown = 0x1p-24f;  // factor of an operand before it is split
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = pack2(a, b);
    const float ra = a - lo2(h), rb = b - hi2(h);
    m = pack2(ra, rb);
    l = pack2(ra - lo2(m), rb - hi2(m));
}
__device__ __forceinline__ float joined(uint32_t h, uint32_t m, uint32_t l) { return lo2(h) + (lo2(m) + lo2(l)); }
// Operand of eight k in NP parts (NP = 1: a bf16 number, without a factor).
template <int NP> struct Parts { bf16x8 p[NP]; };
__device__ __forceinline__ Parts<3> split8(const float* x) {
    u32x4 h, m, l;
    _Pragma("unroll") for (int i = 0; i < 4; ++i) {
        uint32_t a, b, c;
        split2(x[2 * i], x[2 * i + 1], a, b, c);
        h[i] = a; m[i] = b; l[i] = c;
    }
    return Parts<3>{{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)}};
}
// every product but that of the heads, smallest first
template <int NA, int NB, typename Acc>
__device__ __forceinline__ void small_terms(const Parts<NA>& a, const Parts<NB>& b, Acc& c) {
    if constexpr (NA == 3 && NB == 3) {
        c = mfma16(a.p[0], b.p[2], c);
        c = mfma16(a.p[2], b.p[0], c);
        c = mfma16(a.p[1], b.p[1], c);
        c = mfma16(a.p[1], b.p[0], c);
        c = mfma16(a.p[0], b.p[1], c);
    } else if constexpr (NA == 3) {
        c = mfma16(a.p[2], b.p[0], c);
        c = mfma16(a.p[1], b.p[0], c);
    } else if constexpr (NB == 3) {
        c = mfma16(a.p[0], b.p[2], c);
        c = mfma16(a.p[0], b.p[1], c);
    }
}
// Schedule the N matrix instructions of this piece of code with V vector instructions after each: a wave issues in order, and
// an instruction behind two dependent matrix ones waits with the second.
template <int N, int V>
__device__ __forceinline__ void interleave() {
    _Pragma("unroll") for (int i = 0; i < N; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
}
__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= FLT_MAX; }
__device__ __forceinline__ void replace_not_finite(f32x16& x, const f32x16& y) {
    _Pragma("unroll") for (int i = 0; i < 16; ++i) x[i] = finite(x[i]) ? x[i] : y[i];
}
__device__ __forceinline__ float not_finite(const f32x16& x) {  // NaN if any element is infinite or NaN, else 0
    float c = 0.f;
    _Pragma("unroll") for (int i = 0; i < 16; ++i) c = fmaf(x[i], 0.f, c);
    return c;
}

// Rows of the scalar kinds' walker in LDS, part by part.  Keys (and bf16 values) as they come; queries with the four-element
// groups of every 16 features in the order 0, 2, 1, 3, so that the features of result registers 8s .. 8s+7, which an
// operand out of the accumulators has as its k, lie in one 16-byte piece.
// Rows follow one another 16 bytes apart, so that reads of 16 lanes tile the banks, or (XCH, 64-wide rows) without a gap, the
// 16-byte pieces of a row exchanged instead: 16 rows' pieces of one column, and 4 x 32 bytes of 8 rows, lie in different banks.
template <int NP, int RW, bool XCH>
struct GRows {
    static_assert(!XCH || RW == 64, "eight pieces to a row");
    static constexpr int LDR = XCH ? RW : RW + 8, PART = GT * LDR;  // elements
    __device__ static __forceinline__ int pos(int row, int col) {
        return row * LDR + (XCH ? col ^ (((row & 6) | ((row >> 3) & 1)) << 3) : col);
    }
    template <typename TIO, int W, int NT>
    __device__ static __forceinline__ void commit(uint16_t* dst, const GTile<TIO, W, NT>& t, int tid, bool swap) {
        using Tile = GTile<TIO, W, NT>;
        _Pragma("unroll") for (int i = 0; i < Tile::CNT; ++i) {
            const int p = tid + NT * i, row = p / Tile::PR, c = p % Tile::PR;
            const u32x4 x = t.v[i];
            if constexpr (NP == 3) {
                const int q = swap ? (c & ~3) | ((c & 1) << 1) | ((c >> 1) & 1) : c;
                u32x2 h, m, l;
                _Pragma("unroll") for (int e = 0; e < 2; ++e) {
                    uint32_t a, b, d;
                    split2(__uint_as_float(x[2 * e]) * kUp, __uint_as_float(x[2 * e + 1]) * kUp, a, b, d);
                    h[e] = a; m[e] = b; l[e] = d;
                }
                uint16_t* o = dst + pos(row, 4 * q);
                *reinterpret_cast<u32x2*>(o) = h;
                *reinterpret_cast<u32x2*>(o + PART) = m;
                *reinterpret_cast<u32x2*>(o + 2 * PART) = l;
            } else if (swap) {
                const int f = 16 * (c >> 1) + 4 * (c & 1);
                *reinterpret_cast<u32x2*>(dst + pos(row, f)) = u32x2{x.x, x.y};
                *reinterpret_cast<u32x2*>(dst + pos(row, f + 8)) = u32x2{x.z, x.w};
            } else {
                *reinterpret_cast<u32x4*>(dst + pos(row, 8 * c)) = x;
            }
        }
    }
    // element at a stored column (with its factor)
    __device__ static __forceinline__ float at(const uint16_t* src, int row, int col) {
        const uint16_t* o = src + pos(row, col);
        if constexpr (NP == 3) return joined(o[0], o[PART], o[2 * PART]);
        else return lo2(o[0]);
    }
    __device__ static __forceinline__ int swapped(int f) { return (f & ~12) | ((f & 4) << 1) | ((f & 8) >> 1); }
    // eight features of one row: 16 consecutive bytes, or two groups of four elements, 8 apart
    __device__ static __forceinline__ Parts<NP> row8(const uint16_t* src, int row, int col) {
        Parts<NP> r;
        _Pragma("unroll") for (int i = 0; i < NP; ++i) r.p[i] = *reinterpret_cast<const bf16x8*>(src + i * PART + pos(row, col));
        return r;
    }
    __device__ static __forceinline__ Parts<NP> row44(const uint16_t* src, int row, int col) {
        Parts<NP> r;
        _Pragma("unroll") for (int i = 0; i < NP; ++i) {
            const uint16_t* o = src + i * PART;
            const u32x2 a = *reinterpret_cast<const u32x2*>(o + pos(row, col)), b = *reinterpret_cast<const u32x2*>(o + pos(row, col + 8));
            r.p[i] = __builtin_bit_cast(bf16x8, u32x4{a.x, a.y, b.x, b.y});
        }
        return r;
    }
    // one column of rows hrow(8 s + 0 .. 7): the transposing LDS read hands lane i of 16 the i-th feature of a patch of 4 rows
    __device__ static __forceinline__ Parts<NP> col8(const uint16_t* src, int s, int col0, int lane) {
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
        const int r = lane & 15, row = 16 * s + 4 * (lane >> 5) + (r >> 2), col = col0 + 16 * ((lane >> 4) & 1) + 4 * (r & 3);
        Parts<NP> o;
        _Pragma("unroll") for (int i = 0; i < NP; ++i) {
            const uint16_t* p = src + i * PART;
            const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + pos(row, col))));
            const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + pos(row + 8, col))));
            o.p[i] = __builtin_bit_cast(bf16x8, u32x4{a.x, a.y, b.x, b.y});
        }
        return o;
    }
};

// LDS of the scalar kinds' walker, in bytes.  fp32 values are read by columns, a wave's two halves four rows apart, and four
// columns at a time by rows: either 4 * stride == 32 mod 64 words, or (XCH) no gap and 8-column pieces exchanged by the row's bits
// 1 to 3, bit 2 between the halves of the row.
//   Q | K | V | scores: three parts [2][64][8], then the pairs (p, p) | two sets of decay tables | row products
// XCH for fp32, 64 x 64, without helpers: four workgroups fit on a compute unit, the number that the segment plan counts on (with
// gaps 44736 bytes and three, three quarters of a grid and then the rest: forward, 64 sequences of 1024 63 -> 54 us, 1024 of 512
// 219 -> 165; forward + backward, 64 of 1024, 198 -> 177).  With helpers the exchange only costs instructions (23.7 -> 24.3 us for 2
// sequences of 256).
template <typename TIO, int KD, int TV, int HW, bool SUM>
struct GLdsS {
    static constexpr int NP = sizeof(TIO) == 4 ? 3 : 1, NW = TV / 32, NT = 64 * (NW + HW);
    static constexpr bool XCH = NP == 3 && KD == 64 && TV == 64 && HW == 0;
    using Rows = GRows<NP, KD, XCH>;
    static constexpr int LV = XCH ? TV : TV + 8, rows = NP * Rows::PART * 2;
    __device__ static __forceinline__ int vpos(int row, int col) {
        return row * LV + (XCH ? col ^ (((row >> 2) & 1) << 5 | ((row >> 3) & 1) << 4 | ((row >> 1) & 1) << 3) : col);
    }
    static constexpr int oK = SUM ? 0 : rows, oV = oK + rows, oP = oV + GT * LV * int(sizeof(TIO)), oD = oP + (SUM ? 0 : 3 * 2048);
    static constexpr int oT = oD + (SUM ? 0 : GT * 4), table = 34 * 8 + 2 * GT * 4 + 16, oR = oT + 2 * table, bytes = oR + (SUM ? 0 : NW * GT * 8);
};

// Walker of the scalar kinds.  TV / 32 waves, wave w owning value features [32 w, 32 w + 32) of the state, all key features, and
// HW helpers, which take their share of the rows and all of scores and tables.  Two workgroups of the 128-wide form share a
// compute unit (77 KiB of LDS each), and one's matrix work runs under the other's waits.
template <typename TIO, int KD, int TV, int HW, bool SUM>
__global__ __launch_bounds__(2 * TV + 64 * HW, KD == 256 ? 1 : 2) void gk_walk(Dims d, GArgs a) {
    using Lds = GLdsS<TIO, KD, TV, HW, SUM>;
    constexpr int NP = Lds::NP, NW = Lds::NW, NT = Lds::NT, KB = KD / 32;
    // The next rows are requested at the start of a step, but where a wave holds twice as many (two waves to 128-wide keys).
    constexpr bool EARLY = KD == 64 || NT == 256;
    using Rows = typename Lds::Rows;
    using VRows = GRows<1, TV, false>;                      // bf16 values
    extern __shared__ __align__(16) char smb[];
    uint16_t *Q = reinterpret_cast<uint16_t*>(smb), *K = reinterpret_cast<uint16_t*>(smb + Lds::oK), *Pp = reinterpret_cast<uint16_t*>(smb + Lds::oP);
    TIO* V = reinterpret_cast<TIO*>(smb + Lds::oV);
    float* pdv = reinterpret_cast<float*>(smb + Lds::oD);
    double* dred = reinterpret_cast<double*>(smb + Lds::oR);  // [wave][32]: partial row products
    // decay tables of a step: E_p [32] and the step's total, e^{E_p}, 2^24 e^{E - E_p} of all but the last two tokens (0 there)
    // and of those two
    struct Tables { double* bs; float *wi, *wo, *wl; };
    auto tables = [&](int kk) {
        char* t = smb + Lds::oT + (kk & 1) * Lds::table;
        float* f = reinterpret_cast<float*>(t + 34 * 8);
        return Tables{reinterpret_cast<double*>(t), f, f + GT, f + 2 * GT};
    };

    // factors to take out of a product of scores (rows x rows) and of any other (rows x what is split in registers)
    constexpr float kScores = NP == 3 ? kDown * kDown : 1.f, kRows = NP == 3 ? kDown * kDown : kDown;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Every phase reads LDS at its own lane-dependent addresses.  Left alone the compiler keeps them all in registers
    // across the loop (over a hundred); with the thread id hidden at the start of a phase it recomputes that phase's few.
    auto fresh = [&]() { int t = tid; asm volatile("" : "+v"(t)); return t; };
    const int slice = blockIdx.z % a.nsl;
    const GRole& R = a.role[blockIdx.z / a.nsl];
    const int rev = R.rev, vcol = slice * TV;               // first value column of this workgroup
    const GWalk s = find_walk(d, a, rev, SUM);
    if (s.none) return;
    const size_t sz = size_t(a.kd) * a.vd;

    GTile<TIO, KD, NT> rq, rk;
    GTile<TIO, TV, NT> rv;
    auto gload = [&](int kk) {
        const int tid = fresh();
        const ChunkPos p = walk_step(d, s, rev, kk);
        const uint32_t kb = uint32_t(p.ts) * a.kd * sizeof(TIO), vb = uint32_t(p.ts) * a.vd * sizeof(TIO);
        if (!SUM) rq.gload(static_cast<const TIO*>(R.xq) + p.tok0 * a.kd, kb, p.L, rev, tid);
        rk.gload(static_cast<const TIO*>(R.xk) + p.tok0 * a.kd, kb, p.L, rev, tid);
        rv.gload(static_cast<const TIO*>(R.xv) + p.tok0 * a.vd + vcol, vb, p.L, rev, tid);
    };
    // an element of a row as it came, row < L
    auto number = [&](const void* x, const ChunkPos& p, int row, int col) {
        const TIO* e = static_cast<const TIO*>(x) + (p.tok0 + size_t(rev ? p.L - 1 - row : row) * p.ts) * a.kd + col;
        if constexpr (NP == 3) return *e;
        else return lo2(*e);
    };
    // The last wave, which has the fewest score blocks, makes the decay tables, a step ahead of their use.
    const bool tabler = w == NW + HW - 1, carrier = HW == 0 || w < NW;
    double gtot = 0.0;
    // Log-decay of walk position lane % 32.  Every wave loads, and something also where there is none: a branch here would
    // wait for all rows on their way (0 where the tables are made).
    const float* gp = d.kind == 0 ? static_cast<const float*>(R.xk) : d.kind == 1 ? a.g + s.walk.bh % d.H : a.g;
    auto decay_load = [&](int kk) {
        const ChunkPos p = walk_step(d, s, rev, kk);
        const int row = min(fresh() & 31, p.L - 1);
        const float* base = d.kind == 2 ? gp + p.tok0 : gp;
        return base[d.kind == 2 ? uint32_t(rev ? p.L - 1 - row : row) * uint32_t(p.ts) : 0u];
    };
    // E in fp64: the sums reach hundreds for strong decays while only their O(1) differences enter exp()
    auto decay_tables = [&](int kk, float gval) {
        const int lane = fresh() & 63, n = lane & 31;
        const Tables t = tables(kk);
        const int L = walk_step(d, s, rev, kk).L;
        const double x = n < L && d.kind != 0 ? double(gval) : 0.0;
        double inc = x;
        for (int off = 1; off < GT; off <<= 1) {
            const double y = __shfl_up(inc, off, 32);
            if (n >= off) inc += y;
        }
        const double all = __shfl(inc, GT - 1, 32), E = rev ? inc - x : inc;
        if (lane < GT) {
            t.bs[n] = E;
            t.wi[n] = expf(float(E));
            const float wo = expf(float(all - E)) * kUp;
            t.wo[n] = n < L - 2 ? wo : 0.f;
            if (n >= L - 2 && n < L) t.wl[n - (L - 2)] = wo;
            if (n == 0) t.bs[GT] = all;
        }
        gtot += all;
    };
    float gval = 0.f;                                       // of the step after the one whose tables are there
    if (s.cnt > 0) {
        const float g0 = decay_load(0);
        gload(0);
        gval = decay_load(1);
        if (tabler) decay_tables(0, g0);
    }
    f32x16 S[KB];
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib) S[ib] = f32x16{0};
    if (!SUM) {
        const float* e = s.wseg > 0 ? R.bound + bound_at(R.per, s.slot0, s.unit0, s.wseg) * sz : R.edge_in ? R.edge_in + size_t(s.walk.edge) * sz : nullptr;
        if (e && carrier) state_load(S, e, R.trans, a.kd, a.vd, 0, vcol + 32 * w, fresh() & 63);
    }
    if (!SUM)  // the quarter of the score block whose keys follow its queries stays zero
        for (int e = tid; e < 3 * 128; e += NT) *reinterpret_cast<u32x4*>(Pp + (e * 8)) = u32x4{0, 0, 0, 0};

    for (int kk = 0; kk < s.cnt; ++kk) {
        const ChunkPos cp = walk_step(d, s, rev, kk);
        const int L = cp.L;
        const Tables T = tables(kk);
        if (!SUM && carrier && R.dot) {
            const int u = unit_end(d, s, rev, kk);
            if (u >= 0) {
                const int lane = fresh() & 63;
                double z = 0.0;  // (a sequence's last step starts from the edge state)
                if (kk > 0 || s.wseg > 0 || R.edge_in) z = state_dot(S, R.dot + (s.unit0 + u) * sz, a.kd, 0, vcol + 32 * w, lane);
                for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off, 64);
                if (lane == 0) R.z[(s.unit0 + u) * (a.vd / 32) + vcol / 32 + w] = z;
            }
        }
        {
            const int tid = fresh();
            if (!SUM) rq.clear(L, tid);
            rk.clear(L, tid);
            rv.clear(L, tid);
            if (!SUM) Rows::commit(Q, rq, tid, true);
            Rows::commit(K, rk, tid, false);
            if constexpr (NP == 3)
                _Pragma("unroll") for (int i = 0; i < rv.CNT; ++i) {
                    const int p = tid + NT * i;
                    *reinterpret_cast<u32x4*>(V + Lds::vpos(p / rv.PR, 4 * (p % rv.PR))) = rv.v[i];
                }
            else VRows::commit(V, rv, tid, false);
        }
        __syncthreads();  // (A) rows and decay tables of this step are in LDS
        if (EARLY) gload(kk + 1);
        const float gnext = decay_load(kk + 2);
        // this lane's four times four consecutive output features, 8 apart: uniform base + a 32-bit offset
        const size_t obase = cp.tok0 * a.vd + vcol + 32 * w;
        const uint32_t oel = [&] {
            const int l = fresh() & 63, n = min(l & 31, L - 1);
            return uint32_t(rev ? L - 1 - n : n) * (uint32_t(cp.ts) * uint32_t(a.vd)) + 4 * (l >> 5);
        }();
        f32x4 aux[4];                                       // the elements they are multiplied with
        if (!SUM && carrier && R.xdot)  // (a helper has no columns of its own)
            _Pragma("unroll") for (int g = 0; g < 4; ++g) aux[g] = load4(static_cast<const TIO*>(R.aux) + obase + oel + 8 * g);
        f32x16 O;
        if (!SUM) {
            // Blocks of 16 x 16 scores P^T[s][p] = y_s . x_p, keys 16 (b / 2) .., queries 16 ((b + 1) / 2) ..: a block to each of the
            // first three of four waves, or the first two (same keys) to one of two and the third to the other (the helpers, if any).
            if (HW ? !carrier : NW == 2 || w < 3) {
                constexpr int NB = NW == 2 ? 2 : 1;
                const int lane = fresh() & 63, c = lane & 15, q = lane >> 4, b0 = (HW ? w - NW : w) * NB, nb = min(NB, 3 - b0), sb = 16 * (b0 >> 1);
                f32x4 P[NB];
                {   // an accumulator for each of the products: short chains
                    constexpr int NA = NP == 3 ? 6 : 1;
                    f32x4 acc[NB][NA];
                    _Pragma("unroll") for (int b = 0; b < NB; ++b)
                        _Pragma("unroll") for (int i = 0; i < NA; ++i) acc[b][i] = f32x4{0.f, 0.f, 0.f, 0.f};
                    _Pragma("unroll") for (int f = 0; f < KD; f += 32) {
                        const Parts<NP> y = Rows::row44(K, sb + c, f + 16 * (q >> 1) + 4 * (q & 1));
                        _Pragma("unroll") for (int b = 0; b < NB; ++b) {
                            const Parts<NP> x = Rows::row8(Q, 16 * ((min(b0 + b, 2) + 1) >> 1) + c, f + 8 * q);
                            _Pragma("unroll") for (int i = 0; i < NA; ++i) {
                                constexpr int py[6] = {0, 1, 0, 1, 2, 0}, px[6] = {0, 0, 1, 1, 0, 2};
                                acc[b][i] = mfma16(y.p[py[i]], x.p[px[i]], acc[b][i]);
                            }
                        }
                    }
                    _Pragma("unroll") for (int b = 0; b < NB; ++b) {
                        P[b] = acc[b][0];
                        if constexpr (NP == 3) P[b] += (acc[b][1] + acc[b][2]) + (acc[b][3] + (acc[b][4] + acc[b][5]));
                    }
                }
                _Pragma("unroll") for (int b = 0; b < NB; ++b) {
                    if (b >= nb) break;
                    const int p = 16 * ((b0 + b + 1) >> 1) + c;
                    f32x4 t = P[b];
                    const bool again = __any(fmaf(t[0] + t[1], 0.f, (t[2] + t[3]) * 0.f) != 0.f);
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) t[j] *= kScores;
                    if (again) {
                        f32x4 G = {0.f, 0.f, 0.f, 0.f};
                        _Pragma("unroll 1") for (int f = 0; f < KD; ++f) {
                            const float x = number(R.xq, cp, min(p, L - 1), f);
                            _Pragma("unroll") for (int j = 0; j < 4; ++j) G[j] = fmaf(number(R.xk, cp, min(sb + 4 * q + j, L - 1), f), x, G[j]);
                        }
                        _Pragma("unroll") for (int j = 0; j < 4; ++j) t[j] = finite(t[j]) ? t[j] : G[j];
                    }
                    // decayed, in three parts and the order an operand has them; pairs (r < p) only, and (p, p) apart
                    const double bp = T.bs[p];
                    uint32_t h[2], m[2], l[2];
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) {
                        const int r = sb + 4 * q + j;
                        if (r == p) pdv[p] = t[j];
                        if (d.kind != 0) t[j] *= expf(float(bp - T.bs[r]));
                        t[j] = r < p ? t[j] : 0.f;  // (not t * 0: t may be infinite)
                    }
                    const f32x4 u = t * kUp;
                    _Pragma("unroll") for (int j = 0; j < 2; ++j) split2(u[2 * j], u[2 * j + 1], h[j], m[j], l[j]);
                    auto fits = [&](int j) { return fabsf(t[j]) < 0x1p103f; };  // (to 2^104 the head could round to infinity)
                    if (__any(!(fits(0) && fits(1) && fits(2) && fits(3))))     // its bits instead of parts
                        _Pragma("unroll") for (int j = 0; j < 4; ++j)
                            if (!fits(j)) {
                                const uint32_t word = __float_as_uint(t[j]), at = 16 * (j & 1), keep = 0xffff0000u >> at;
                                h[j >> 1] = (h[j >> 1] & keep) | (0x7f80u << at);
                                m[j >> 1] = (m[j >> 1] & keep) | ((word >> 16) << at);
                                l[j >> 1] = (l[j >> 1] & keep) | ((word & 0xffffu) << at);
                            }
                    uint16_t* o = Pp + ((sb >> 4) * 64 + (q & 1) * 32 + p) * 8 + 4 * (q >> 1);
                    *reinterpret_cast<u32x2*>(o) = u32x2{h[0], h[1]};
                    *reinterpret_cast<u32x2*>(o + 1024) = u32x2{m[0], m[1]};
                    *reinterpret_cast<u32x2*>(o + 2048) = u32x2{l[0], l[1]};
                }
            }
            if (tabler && kk + 1 < s.cnt) decay_tables(kk + 1, gval);
            if (carrier) {  // inter: O^T[v][p] = e^{E_p} sum_i S[i][v] x_p[i], the state blocks as A operands out of the accumulators
                const int lane = fresh() & 63, n = lane & 31, half = lane >> 5;
                f32x16 small = {0};
                O = f32x16{0};
                _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                        float t[8];
                        _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = S[ib][8 * h + x] * kUp;
                        const Parts<3> sp = split8(t);
                        const Parts<NP> x = Rows::row8(Q, n, 32 * ib + 16 * h + 8 * half);
                        small_terms(sp, x, small);
                        O = mfma16(sp.p[0], x.p[0], O);
                    }
                interleave<KB * 2 * (NP == 3 ? 6 : 3), NP == 3 ? 8 : 16>();
                _Pragma("unroll") for (int x = 0; x < 16; ++x) O[x] += small[x];
                const float nf = not_finite(O), e = T.wi[n];
                _Pragma("unroll") for (int x = 0; x < 16; ++x) O[x] *= kRows;
                if (__any(nf != nf)) {
                    f32x16 G = {0};
                    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
                        _Pragma("unroll") for (int x = 0; x < 16; ++x)
                            G = mfma2(S[ib][x], number(R.xq, cp, min(n, L - 1), 32 * ib + hrow(x, half)), G);
                    replace_not_finite(O, G);
                }
                _Pragma("unroll") for (int x = 0; x < 16; ++x) O[x] *= e;
            }
            __syncthreads();  // (B) scores
            if (carrier) {
                const int lane = fresh() & 63, n = lane & 31, half = lane >> 5;
                // intra: X[v][p] = sum_s Z[s][v] P[s][p].  P is zero where s does not precede p, but a zero times an infinity or NaN is
                // not: a value row that is not finite would reach the positions before it, which must not depend on it.  Then the
                // product runs without such elements and they are added pair by pair.
                f32x16 X;
                float xs = kRows;                           // the factor to take out of X
                {
                    Parts<3> pp[2];
                    _Pragma("unroll") for (int h = 0; h < 2; ++h)
                        _Pragma("unroll") for (int i = 0; i < 3; ++i) pp[h].p[i] = *reinterpret_cast<const bf16x8*>(Pp + i * 1024 + (h * 64 + lane) * 8);
                    auto product = [&](auto&& part) {
                        X = f32x16{0};
                        Parts<NP> vp[2];
                        _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                            vp[h] = part(h);
                            small_terms(vp[h], pp[h], X);
                        }
                        _Pragma("unroll") for (int h = 0; h < 2; ++h) X = mfma16(vp[h].p[0], pp[h].p[0], X);
                    };
                    auto value = [&](int row, int col) { if constexpr (NP == 3) return V[Lds::vpos(row, col)]; else return lo2(V[Lds::vpos(row, col)]); };
                    product([&](int h) {
                        if constexpr (NP == 3) {
                            float t[8];
                            _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = V[Lds::vpos(hrow(8 * h + x, half), 32 * w + n)] * kUp;
                            return split8(t);
                        } else {
                            return VRows::col8(V, h, 32 * w, lane);
                        }
                    });
                    const float nf = not_finite(X);
                    if (__any(nf != nf)) {
                        auto known = [&](int x) { const float t = value(hrow(x, half), 32 * w + n); return finite(t) ? t : 0.f; };
                        auto score = [&](int r, int p) {
                            const uint16_t* o = Pp + ((r >> 4) * 64 + ((r >> 2) & 1) * 32 + p) * 8 + 4 * ((r >> 3) & 1) + (r & 3);
                            return (o[0] & 0x7f80) == 0x7f80 ? __uint_as_float(uint32_t(o[1024]) << 16 | o[2048]) : joined(o[0], o[1024], o[2048]) * kDown;
                        };
                        product([&](int h) {
                            float t[8];
                            _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = known(8 * h + x);
                            if constexpr (NP == 3) {
                                _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] *= kUp;
                                return split8(t);
                            } else return Parts<1>{{__builtin_bit_cast(bf16x8, u32x4{pack2(t[0], t[1]), pack2(t[2], t[3]), pack2(t[4], t[5]), pack2(t[6], t[7])})}};
                        });
                        f32x16 G = {0};
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) G = mfma2(known(x), score(hrow(x, half), n), G);
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) X[x] *= kRows;
                        xs = 1.f;
                        replace_not_finite(X, G);
                        _Pragma("unroll 1") for (int r = 0; r < GT; ++r) {
                            const float p = score(r, n);
                            _Pragma("unroll") for (int x = 0; x < 16; ++x) {
                                const float t = value(r, 32 * w + hrow(x, half));
                                if (r < n && !finite(t)) X[x] += t * p;
                            }
                        }
                    }
                }
                // The pair (p, p) stays out of the product with aux: it is the same number in q.dq and in k.dk and cancels in the
                // decay gradient, exactly instead of to rounding.
                const float pd = pdv[n];
                double t = 0.0;
                _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                    f32x4 o;
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) o[j] = fmaf(X[4 * g + j], xs, O[4 * g + j]);
                    if (R.xdot) {
                        _Pragma("unroll") for (int j = 0; j < 4; ++j) t += double(aux[g][j]) * double(o[j]);
                    }
                    const f32x4 z = load4(V + Lds::vpos(n, 32 * w + 8 * g + 4 * half));
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) o[j] += pd * z[j];
                    if (n < L) store4(static_cast<TIO*>(R.out) + obase + oel + 8 * g, o);
                }
                if (R.xdot) {
                    t += __shfl_xor(t, 32, 64);
                    if (half == 0) dred[w * GT + n] = t;
                }
            }
        } else if (tabler && kk + 1 < s.cnt) {
            decay_tables(kk + 1, gval);
        }
        if (!EARLY) gload(kk + 1);
        if (carrier) {  // S[i][v] = e^E S[i][v] + sum_t e^{E - E_t} y_t[i] z_t[v]; the step's own sum is formed by itself, so the state sees
            // one rounding per step instead of one per token.  The latest tokens, which weigh most, come last, and the last two
            // as they are: in parts the large product would be rounded once by itself and once with the small ones (final state
            // under a strong decay 3.8e-8 instead of 2.7e-8).
            const int lane = fresh() & 63, n = lane & 31, half = lane >> 5;
            Parts<3> z[2];
            _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                float t[8];
                const f32x4 e0 = *reinterpret_cast<const f32x4*>(T.wo + 16 * h + 4 * half), e1 = *reinterpret_cast<const f32x4*>(T.wo + 16 * h + 8 + 4 * half);
                if constexpr (NP == 3) {
                    _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = V[Lds::vpos(hrow(8 * h + x, half), 32 * w + n)];
                } else {
                    const u32x4 r = __builtin_bit_cast(u32x4, VRows::col8(V, h, 32 * w, lane).p[0]);
                    _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = x & 1 ? hi2(r[x >> 1]) : lo2(r[x >> 1]);
                }
                _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] *= x < 4 ? e0[x & 3] : e1[x & 3];
                z[h] = split8(t);
            }
            auto weight = [&](int r) { return r < L - 2 ? T.wo[r] : r < L ? T.wl[r - (L - 2)] : 0.f; };
            auto value = [&](int r) { if constexpr (NP == 3) return V[Lds::vpos(r, 32 * w + n)]; else return lo2(V[Lds::vpos(r, 32 * w + n)]); };
            const int last = L - 2 + half < 0 ? GT - 1 : L - 2 + half;  // (one token: with a row of zeros)
            const float zlast = value(last) * weight(last);
            const float lam = expf(float(T.bs[GT]));
            constexpr int GB = SUM && EARLY && KB >= 4 ? 4 : 2;  // blocks at a time: independent chains, one look for what is not finite
            _Pragma("unroll") for (int i0 = 0; i0 < KB; i0 += GB) {
                f32x16 U[GB];
                _Pragma("unroll") for (int b = 0; b < GB; ++b) {
                    const int i = 32 * (i0 + b);
                    U[b] = f32x16{0};
                    Parts<NP> y[2];
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                        y[h] = Rows::col8(K, h, i, lane);
                        small_terms(y[h], z[h], U[b]);
                    }
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) U[b] = mfma16(y[h].p[0], z[h].p[0], U[b]);
                    U[b] = mfma2(Rows::at(K, last, i + n), zlast, U[b]);
                }
                float nf = 0.f;
                _Pragma("unroll") for (int b = 0; b < GB; ++b) {
                    nf += not_finite(U[b]);
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) U[b][x] *= kRows;
                }
                if (__any(nf != nf)) {
                    _Pragma("unroll") for (int b = 0; b < GB; ++b) {
                        f32x16 G = {0};
                        _Pragma("unroll 1") for (int x = 0; x < 16; ++x) {
                            const int r = 2 * x + half;
                            const float y = number(R.xk, cp, min(r, L - 1), 32 * (i0 + b) + n);
                            G = mfma2(r < L ? y : 0.f, value(r) * (weight(r) * kDown), G);
                        }
                        replace_not_finite(U[b], G);
                    }
                }
                _Pragma("unroll") for (int b = 0; b < GB; ++b)
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) S[i0 + b][x] = fmaf(lam, S[i0 + b][x], U[b][x]);
            }
        }
        gval = gnext;
        if (!SUM) {
            const long long u = keep_slot(d, R, s, kk);
            if (u >= 0 && carrier) state_store(S, R.bound + u * sz, R.trans, a.kd, a.vd, 0, vcol + 32 * w, fresh() & 63);
        }
        __syncthreads();  // (D) every read of this step's tiles is done
        if (!SUM && R.xdot && tid < L) {
            double t = 0.0;
            _Pragma("unroll") for (int u = 0; u < NW; ++u) t += dred[u * GT + tid];
            R.xdot[size_t(slice) * d.BH() * d.T + cp.wtok0 + (rev ? L - 1 - tid : tid)] = float(t);
        }
    }

    float* e = nullptr;
    if (SUM) e = R.bound + bound_at(R.per, s.slot0, s.unit0, s.wseg + 1) * sz;
    else if (s.empty || s.wseg == s.nsq - 1) e = R.edge_out ? R.edge_out + size_t(s.walk.edge) * sz : nullptr;
    if (e && carrier) state_store(S, e, R.trans, a.kd, a.vd, 0, vcol + 32 * w, fresh() & 63);
    if (SUM && slice == 0 && d.kind != 0 && tabler && (tid & 63) == 0) R.gseg[s.slot0 + s.wseg] = gtot;
}

// Walker of the vector kind.  VEC 1: a decay per key-role feature (o, dv: the scores carry the decay).  VEC 2: a decay per
// value-role feature (dq, dk: the outputs do).
//
// The pair weights e^{E_p - E_s} do not factor over the pair, but split at a reference between s and p they
// do, into two factors <= 1.  At level l = 16, 8, 4, 2, 1 the pairs whose positions first differ in bit log2 l are taken
// together (p in an odd block of l positions, s in the even block before it, reference at the start of p's block): every
// position is on one side only, so one tile W holds, row by row, either side's weighted operand.  Running sums start at
// the reference, so they are exact where the weight matters, however strong the decay.
//
// Two groups of TV / 32 waves; wave w of either group owns value features [32 w, 32 w + 32) and half of the key features:
//   lead  the score blocks, what is done with them, and the output;
//   aux   the rows (requested a step ahead) and the weighted tiles (a phase ahead).
// Both hold their half of the state, form its part of the inter product and move it on, so that the vector work of one
// group runs under the matrix work of the other (one group doing both in turn, gradient walks of d_k = 64, d_v = 128, bf16,
// 4 x 8 sequences of 2048: 0.260 ms; this: 0.171).  Each group runs a loop of its own with the same barriers, which the
// comments of both number.
template <typename TIO, int KD, int TV, int VEC, bool SUM>
__global__ __launch_bounds__(4 * TV, KD == 256 ? 1 : 2) void gk_walk_vec(Dims d, GArgs a) {
    using Lds = GLds<TIO, KD, TV, VEC, SUM>;
    constexpr bool RAW = Lds::RAW;
    using KRows = GRows<1, KD, false>;  // bf16 rows as they came: queries with the groups of four exchanged, keys and values in order
    using VRows = GRows<1, TV, false>;
    constexpr int NW = Lds::NW, NT = 2 * TV, LQ = Lds::LQ, LV = Lds::LV, KB = KD / 64, COLS = Lds::COLS, LW = COLS + 4;
    constexpr int PIECES = Lds::PIECES, LEN = GT / PIECES, ITEMS = (PIECES * COLS + NT - 1) / NT;
    extern __shared__ __align__(16) float sm[];
    float *Q = sm, *K = sm + Lds::oK, *V = sm + Lds::oV, *Pp = sm + Lds::oP, *W0 = sm + Lds::oW, *W1 = W0 + Lds::WT;
    uint16_t *Qb = reinterpret_cast<uint16_t*>(Q), *Kb = reinterpret_cast<uint16_t*>(K), *Vb = reinterpret_cast<uint16_t*>(V);
    // element of a value or key row, as the kernel has them
    auto value = [&](int row, int col) { if constexpr (RAW && VEC == 1) return VRows::at(Vb, row, col); else return V[row * LV + col]; };
    auto key = [&](int row, int col) { if constexpr (RAW && VEC == 2) return KRows::at(Kb, row, col); else return K[row * LQ + col]; };
    double* tot = reinterpret_cast<double*>(sm + Lds::oT);  // log-decay of the pieces of the step [PIECES][COLS]
    float* lamv = sm + Lds::oT + 2 * PIECES * COLS;         // e^E [COLS]
    float *fwdp = lamv + COLS, *bwdp = fwdp + 4 * COLS;     // four pieces: products of a piece's decays from either end [4][COLS]

    // the wave index as a scalar: the branch between the groups is then a scalar branch
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave % NW;
    const bool aux = wave >= NW;
    const int tid = threadIdx.x & (NT - 1);                 // index within the group
    // (as in gk_walk)
    auto fresh = [&]() { int t = tid; asm volatile("" : "+v"(t)); return t; };
    const int slice = blockIdx.z % a.nsl;
    const GRole& R = a.role[blockIdx.z / a.nsl];
    const int rev = R.rev, vcol = slice * TV;               // first value column of this workgroup
    const int kcol = aux ? KD / 2 : 0;                      // first key feature of this group
    const GWalk s = find_walk(d, a, rev, SUM);
    if (s.none) return;
    const size_t sz = size_t(a.kd) * a.vd;
    f32x16 S[KB];
    _Pragma("unroll") for (int ib = 0; ib < KB; ++ib) S[ib] = f32x16{0};
    if (!SUM) {
        const float* e = s.wseg > 0 ? R.bound + bound_at(R.per, s.slot0, s.unit0, s.wseg) * sz : R.edge_in ? R.edge_in + size_t(s.walk.edge) * sz : nullptr;
        if (e) state_load(S, e, R.trans, a.kd, a.vd, kcol, vcol + 32 * w, fresh() & 63);
    }

    // ---- work that both groups do
    // this wave's part of the inter product, O^T[v][p] = sum_i S[i][v] x_p[i], the state blocks as A operands out of the
    // accumulators; bf16 rows as they came (VEC 2): the state in three parts, as the scalar kinds have it.  (bf16, d_k = 64, d_v = 128,
    // 4 x 8 sequences of 2048, the dq and dk walkers with fp32 instructions 80 us; with this, the update's weighted values in
    // parts, the scores' products single and the levels' empty rows left out 63; distance of dg to 64 bits 3.2e-7 -> 2.4e-7.  For o
    // and dv, where rows are weighted too, the split costs what it saves: 77 -> 94 us, not done; the summary 38 -> 37.)
    auto inter = [&](const float* X, int ld) {
        const int l = fresh() & 63, n = l & 31, half = l >> 5;
        f32x16 o = {0};
        auto exact = [&]() {
            f32x16 o = {0};
            _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
                _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                    f32x4 x;
                    const int c = kcol + 32 * ib + 8 * g + 4 * half;
                    if constexpr (RAW && VEC == 2) {
                        _Pragma("unroll") for (int j = 0; j < 4; ++j) x[j] = KRows::at(Qb, n, KRows::swapped(c + j));
                    } else x = *reinterpret_cast<const f32x4*>(X + n * ld + c);
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) o = mfma2(S[ib][4 * g + j], x[j], o);
                }
            return o;
        };
        if constexpr (RAW && VEC == 2) {
            f32x16 small = {0};
            _Pragma("unroll") for (int ib = 0; ib < KB; ++ib)
                _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                    float t[8];
                    _Pragma("unroll") for (int x = 0; x < 8; ++x) t[x] = S[ib][8 * h + x] * kUp;
                    const Parts<3> sp = split8(t);
                    const Parts<1> x = KRows::row8(Qb, n, kcol + 32 * ib + 16 * h + 8 * half);
                    small_terms(sp, x, small);
                    o = mfma16(sp.p[0], x.p[0], o);
                }
            _Pragma("unroll") for (int x = 0; x < 16; ++x) o[x] += small[x];
            const float nf = not_finite(o);
            _Pragma("unroll") for (int x = 0; x < 16; ++x) o[x] *= kDown;
            if (__any(nf != nf)) replace_not_finite(o, exact());
            return o;
        } else {
            return exact();
        }
    };
    // ... and its weight e^{E_p} (VEC 2; VEC 1 has it in the rows)
    auto scale_inter = [&](f32x16& O) {
        const int l = fresh() & 63, n = l & 31, half = l >> 5;
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            const f32x4 e = *reinterpret_cast<const f32x4*>(W0 + n * LW + 32 * w + 8 * g + 4 * half);
            _Pragma("unroll") for (int j = 0; j < 4; ++j) O[4 * g + j] *= e[j];
        }
    };
    // S[i][v] = lam S[i][v] + sum_t Y[t][i] (w_t Z[t][v]); the step's own sum is formed by itself, so the state sees one
    // rounding per step instead of one per token (tokens in order, the latest, which weigh most, last: what is added to them would
    // round them again).  bf16 elements: the weighted side in three parts, the last two tokens apart, as the scalar kinds have it.
    auto update = [&](int L) {
        auto left = [&](int t, int i) { if constexpr (VEC == 1) return W0[t * LW + i]; else return key(t, i); };
        auto right = [&](int t, int v) { if constexpr (VEC == 2) return W0[t * LW + v]; else return value(t, v); };
        float lam = 1.f;
        if (VEC == 2) lam = lamv[32 * w + (fresh() & 31)];
        Parts<3> zp[2];                                     // VEC 2: this wave's weighted values
        auto weighted = [&](const float* col, int h, int half) {  // eight tokens of a column of W0, the last two of the step left out
            float t[8];
            _Pragma("unroll") for (int x = 0; x < 8; ++x) {
                const int r = hrow(8 * h + x, half);
                t[x] = r < L - 2 ? col[r * LW] * kUp : 0.f;
            }
            return split8(t);
        };
        if constexpr (RAW && VEC == 2) {
            const int l = fresh() & 63;
            _Pragma("unroll") for (int h = 0; h < 2; ++h) zp[h] = weighted(W0 + 32 * w + (l & 31), h, l >> 5);
        }
        _Pragma("unroll") for (int ib = 0; ib < KB; ++ib) {
            const int l = fresh() & 63, n = l & 31, half = l >> 5;
            f32x16 U = {0};
            auto exact = [&]() {
                f32x16 U = {0};
                _Pragma("unroll") for (int x = 0; x < 16; ++x) U = mfma2(left(2 * x + half, kcol + 32 * ib + n), right(2 * x + half, 32 * w + n), U);
                return U;
            };
            if constexpr (RAW) {
                if constexpr (VEC == 1) {
                    Parts<3> yp[2];
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                        yp[h] = weighted(W0 + kcol + 32 * ib + n, h, half);
                        const Parts<1> v = VRows::col8(Vb, h, 32 * w, l);
                        small_terms(yp[h], v, U);
                    }
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) U = mfma16(yp[h].p[0], VRows::col8(Vb, h, 32 * w, l).p[0], U);
                } else {
                    Parts<1> y[2];
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                        y[h] = KRows::col8(Kb, h, kcol + 32 * ib, l);
                        small_terms(y[h], zp[h], U);
                    }
                    _Pragma("unroll") for (int h = 0; h < 2; ++h) U = mfma16(y[h].p[0], zp[h].p[0], U);
                }
                const int last = L - 2 + half < 0 ? GT - 1 : L - 2 + half;  // (one token: with a row of zeros)
                const float y = left(last, kcol + 32 * ib + n), z = right(last, 32 * w + n);
                U = mfma2(VEC == 1 ? y * kUp : y, VEC == 2 ? z * kUp : z, U);
                const float nf = not_finite(U);
                _Pragma("unroll") for (int x = 0; x < 16; ++x) U[x] *= kDown;
                if (__any(nf != nf)) replace_not_finite(U, exact());
            } else {
                U = exact();
            }
            _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                f32x4 m = {lam, lam, lam, lam};
                if (VEC == 1) m = *reinterpret_cast<const f32x4*>(lamv + kcol + 32 * ib + 8 * g + 4 * half);
                _Pragma("unroll") for (int j = 0; j < 4; ++j) S[ib][4 * g + j] = fmaf(m[j], S[ib][4 * g + j], U[4 * g + j]);
            }
        }
    };
    // the product with the other direction's state at the unit end that the kk-th step starts from
    auto unit_dot = [&](int kk) {
        if (SUM || VEC != 2 || !R.dot) return;
        const int u = unit_end(d, s, rev, kk);
        if (u < 0) return;
        const int l = fresh() & 63;
        double z = 0.0;
        if (kk > 0 || s.wseg > 0 || R.edge_in) z = state_dot(S, R.dot + (s.unit0 + u) * sz, a.kd, kcol, vcol + 32 * w, l);
        z += __shfl_xor(z, 32, 64);
        if (l < 32) R.z[((s.unit0 + u) * 2 + (aux ? 1 : 0)) * a.vd + vcol + 32 * w + l] = z;
    };
    auto unit_keep = [&](int kk) {
        if (SUM || VEC != 2) return;
        const long long u = keep_slot(d, R, s, kk);
        if (u >= 0) state_store(S, R.bound + u * sz, R.trans, a.kd, a.vd, kcol, vcol + 32 * w, fresh() & 63);
    };
    auto block_store = [&](const f32x16& P) {  // a block of registers to this wave's place among the partials
        const int lane = fresh() & 63;
        _Pragma("unroll") for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(Pp + w * 1024 + (g * 64 + lane) * 4) = f32x4{P[4 * g], P[4 * g + 1], P[4 * g + 2], P[4 * g + 3]};
    };
    // levels alternate between the two tiles: f(level, tile, other tile)
    auto levels = [&](auto f) {
        f(std::integral_constant<int, 16>{}, W1, W0);
        f(std::integral_constant<int, 8>{}, W0, W1);
        f(std::integral_constant<int, 4>{}, W1, W0);
        f(std::integral_constant<int, 2>{}, W0, W1);
        f(std::integral_constant<int, 1>{}, W1, W0);
    };

    if (aux) {
        GTile<TIO, KD, NT> rq, rk;
        GTile<TIO, TV, NT> rv;
        // item = (column, piece): the transitions d_p INTO the positions of its piece and, last piece, the closing
        // one.  Forward: the decay of the token itself; backward: that of the position before.
        float dt[ITEMS][LEN], at[ITEMS][LEN], dn[ITEMS][LEN], closing[ITEMS], closing_n[ITEMS];
        double gtot[ITEMS];
        _Pragma("unroll") for (int i = 0; i < ITEMS; ++i) gtot[i] = 0.0;
        auto item_ok = [&](int t, int i) { return PIECES * COLS >= NT * (i + 1) || t + NT * i < PIECES * COLS; };
        auto item_col = [&](int t, int i) { return (t + NT * i) % COLS; };
        auto item_piece = [&](int t, int i) { return (t + NT * i) / COLS; };
        // (Two pieces have forms of their own: that a piece number is then 0 or 1 is not known to the compiler, and the
        // general ones spill 14 to 28 registers more with 256 decayed features; fp32, d_v = 64, 4 x 8 sequences of 2048, forward 507 us, so
        // and with the outputs formed() 486; d_k = 128 311 and 306.)

        auto gload = [&](int kk) {
            const int tid = fresh();
            const ChunkPos p = walk_step(d, s, rev, kk);
            const uint32_t kb = uint32_t(p.ts) * a.kd * sizeof(TIO), vb = uint32_t(p.ts) * a.vd * sizeof(TIO);
            if (!SUM) rq.gload(static_cast<const TIO*>(R.xq) + p.tok0 * a.kd, kb, p.L, rev, tid);
            rk.gload(static_cast<const TIO*>(R.xk) + p.tok0 * a.kd, kb, p.L, rev, tid);
            rv.gload(static_cast<const TIO*>(R.xv) + p.tok0 * a.vd + vcol, vb, p.L, rev, tid);
            {
                const char* gb = reinterpret_cast<const char*>(a.g + p.tok0 * d.dk + (VEC == 2 ? vcol : 0));
                const uint32_t grow = uint32_t(p.ts) * d.dk * 4;
                _Pragma("unroll") for (int i = 0; i < ITEMS; ++i) {
                    if (!item_ok(tid, i)) continue;
                    const uint32_t col = 4 * item_col(tid, i);
                    const int p0 = LEN * item_piece(tid, i);
                    _Pragma("unroll") for (int x = 0; x < LEN; ++x) {  // (what does not exist is zeroed when it is used)
                        const int pos = p0 + x - rev, tok = min(max(rev ? p.L - 1 - pos : pos, 0), p.L - 1);
                        dn[i][x] = *reinterpret_cast<const float*>(gb + uint32_t(tok) * grow + col);
                    }
                    closing_n[i] = *reinterpret_cast<const float*>(gb + col);
                }
            }
        };
        auto commit = [&](int L) {  // registers of this step -> LDS; decay tables
            const int tid = fresh();
            if constexpr (RAW && VEC == 2) {
                rq.clear(L, tid);
                rk.clear(L, tid);
                KRows::commit(Qb, rq, tid, true);
                KRows::commit(Kb, rk, tid, false);
            } else {
                if (!SUM) rq.commit(Q, LQ, L, tid);
                rk.commit(K, LQ, L, tid);
            }
            if constexpr (RAW && VEC == 1) {
                rv.clear(L, tid);
                VRows::commit(Vb, rv, tid, false);
            } else {
                rv.commit(V, LV, L, tid);
            }
            {
                _Pragma("unroll") for (int i = 0; i < ITEMS; ++i) {
                    if (!item_ok(tid, i)) continue;
                    const int h = item_piece(tid, i);
                    double t = 0.0;
                    _Pragma("unroll") for (int x = 0; x < LEN; ++x) {
                        const int pos = LEN * h + x - rev;
                        dt[i][x] = pos >= 0 && pos < L ? dn[i][x] : 0.f;
                        if (!SUM) at[i][x] = expf(dt[i][x]);
                        t += double(dt[i][x]);
                    }
                    closing[i] = rev && L == GT && (PIECES == 2 ? h != 0 : h == PIECES - 1) ? closing_n[i] : 0.f;
                    tot[h * COLS + item_col(tid, i)] = t + double(closing[i]);
                    if constexpr (!SUM && PIECES == 4) {
                        float f = 1.f, b = 1.f;
                        _Pragma("unroll") for (int x = 0; x < LEN; ++x) f *= at[i][x];
                        _Pragma("unroll") for (int x = LEN - 1; x >= 0; --x) b *= at[i][x];
                        fwdp[h * COLS + item_col(tid, i)] = f;
                        bwdp[h * COLS + item_col(tid, i)] = b;
                    }
                }
            }
        };
        // ---- vector kind: writers of the weighted tiles (see the level scheme above)
        auto each = [&](auto&& f) {  // f(item, piece, column)
            const int tid = fresh();
            _Pragma("unroll") for (int i = 0; i < ITEMS; ++i) {
                if (!item_ok(tid, i)) continue;
                f(i, item_piece(tid, i), item_col(tid, i));
            }
        };
        auto write_start = [&](float* o) {  // weight e^{E_p} from the start of the step; also e^E
            each([&](int i, int h, int c) {
                const double t0 = tot[c];
                double all = 0.0, e = h ? t0 : 0.0;
                if constexpr (PIECES == 4) {
                    e = 0.0;
                    _Pragma("unroll") for (int u = 0; u < PIECES; ++u) {
                        const double t = tot[u * COLS + c];
                        if (u < h) e += t;
                        all += t;
                    }
                }
                _Pragma("unroll") for (int x = 0; x < LEN; ++x) {
                    e += double(dt[i][x]);
                    const int p = LEN * h + x;
                    const float wt = expf(float(e));
                    o[p * LW + c] = VEC == 1 ? Q[p * LQ + c] * wt : wt;
                }
                if (h == 0) lamv[c] = expf(float(PIECES == 4 ? all : t0 + tot[COLS + c]));
            });
        };
        auto write_end = [&](float* o) {  // weight e^{E - E_p} to the end of the step, on the state update's operand
            each([&](int i, int h, int c) {
                double e;
                if constexpr (PIECES == 2) {
                    e = h ? double(closing[i]) : tot[COLS + c];
                } else {
                    e = 0.0;
                    _Pragma("unroll") for (int u = PIECES - 1; u > 0; --u)
                        if (u > h) e += tot[u * COLS + c];
                    if (h == PIECES - 1) e = double(closing[i]);
                }
                if (SUM && h == 0) {
                    const double all = tot[c] + e;
                    lamv[c] = expf(float(all));
                    gtot[i] += all;
                }
                _Pragma("unroll") for (int x = LEN - 1; x >= 0; --x) {
                    const int p = LEN * h + x;
                    o[p * LW + c] = (VEC == 1 ? K[p * LQ + c] : V[p * LV + c]) * expf(float(e));
                    e += double(dt[i][x]);
                }
            });
        };
        // Products of at most 16 decays, from the reference outwards: a rounding per factor, where one exponential of the pair's
        // difference has one for all and a rounded argument under strong decays.  Results are no further from 64 bits for it (512
        // tokens, log-decays of -1e-3 to -20 a token: o and dv 0.4 to 0.9, dq and dk 0.5 to 1.0 times the error with exponentials).
        auto write_level = [&](float* o, auto lvc) {
            constexpr int lv = decltype(lvc)::value;
            each([&](int i, int h, int c) {
                constexpr int B = lv < LEN ? lv : LEN;      // positions of a block in this piece
                _Pragma("unroll") for (int b = 0; b < LEN; b += B) {
                    const int first = LEN * h + b;
                    const bool odd = PIECES == 2 && lv == 16 ? h != 0 : B == lv && LEN % (2 * lv) == 0 ? ((b / lv) & 1) != 0 : ((first / lv) & 1) != 0;
                    float e[B], prod = 1.f;
                    if (lv > LEN && (h & 1) == (odd ? 1 : 0)) prod = odd ? fwdp[(h - 1) * COLS + c] : bwdp[(h + 1) * COLS + c];
                    if (odd) {  // query side: from the block's start up to the position
                        _Pragma("unroll") for (int x = 0; x < B; ++x) { prod *= at[i][b + x]; e[x] = prod; }
                    } else {    // key side: from the position to the block's end
                        _Pragma("unroll") for (int x = B - 1; x >= 0; --x) { e[x] = prod; prod *= at[i][b + x]; }
                    }
                    _Pragma("unroll") for (int x = 0; x < B; ++x) {
                        const int p = first + x;
                        if (VEC == 1) o[p * LW + c] = (odd ? Q[p * LQ + c] : K[p * LQ + c]) * e[x];
                        else o[p * LW + c] = odd ? e[x] : V[p * LV + c] * e[x];
                    }
                }
            });
        };

        if (s.cnt > 0) gload(0);
        for (int kk = 0; kk < s.cnt; ++kk) {
            unit_dot(kk);
            const int L = walk_step(d, s, rev, kk).L;
            commit(L);
            __syncthreads();  // (A) rows and decay tables of this step are in LDS
            gload(kk + 1);
            if constexpr (SUM) {
                write_end(W0);
                __syncthreads();  // (B)
                update(L);
            } else if constexpr (VEC == 1) {
                write_start(W0);
                __syncthreads();  // (B) e^{E_p} x_p
                const f32x16 O = inter(W0, LW);
                write_level(W1, std::integral_constant<int, 16>{});
                __syncthreads();  // (B2)
                levels([&](auto lvc, float*, float* nxt) {
                    constexpr int lv = decltype(lvc)::value;
                    if constexpr (lv > 1) write_level(nxt, std::integral_constant<int, lv / 2>{});
                    else write_end(nxt);
                    __syncthreads();  // (L) next level's tile; after the last: score partials, weighted keys
                });
                __syncthreads();  // (M) the partials are spent
                block_store(O);
                update(L);
            } else {
                write_start(W0);
                write_level(W1, std::integral_constant<int, 16>{});
                f32x16 O = inter(Q, LQ);
                __syncthreads();  // (B) score partials, first tiles
                scale_inter(O);
                __syncthreads();  // (B2) the partials and the first tile are spent
                block_store(O);
                levels([&](auto lvc, float*, float* nxt) {
                    constexpr int lv = decltype(lvc)::value;
                    if constexpr (lv > 1) write_level(nxt, std::integral_constant<int, lv / 2>{});
                    else write_end(nxt);
                    __syncthreads();  // (L) next level's tile; after the last: weighted values
                });
                update(L);
            }
            unit_keep(kk);
            __syncthreads();  // (C) every read of this step's tiles is done
        }
        if (SUM && slice == 0) {
            _Pragma("unroll") for (int i = 0; i < ITEMS; ++i)
                if (item_ok(tid, i) && item_piece(tid, i) == 0) R.gseg[(s.slot0 + s.wseg) * COLS + item_col(tid, i)] = gtot[i];
        }
    } else {
        // this wave's share (a range of features) of the block P^T[s][p] = y_s . x_p
        auto score_part = [&](const float* Y, const float* X, int ld) {
            const int l = fresh() & 63, n = l & 31, half = l >> 5;
            f32x16 P = {0};
            _Pragma("unroll") for (int f = 0; f < KD / NW; f += 8) {
                const int c = w * (KD / NW) + f + 4 * half;
                const f32x4 y = *reinterpret_cast<const f32x4*>(Y + n * ld + c), x = *reinterpret_cast<const f32x4*>(X + n * ld + c);
                _Pragma("unroll") for (int j = 0; j < 4; ++j) P = mfma2(y[j], x[j], P);
            }
            return P;
        };
        // the same from bf16 rows as they came: every product exact
        auto score_raw = [&]() {
            const int l = fresh() & 63, n = l & 31, half = l >> 5;
            f32x16 P = {0};
            _Pragma("unroll") for (int f = 0; f < KD / NW; f += 16) {
                const int c = w * (KD / NW) + f;
                P = mfma16(KRows::row44(Kb, n, c + 4 * half).p[0], KRows::row8(Qb, n, c + 8 * half).p[0], P);
            }
            return P;
        };
        auto part_sum = [&]() {
            const int lane = fresh() & 63;
            f32x16 P;
            _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                f32x4 t = *reinterpret_cast<const f32x4*>(Pp + (g * 64 + lane) * 4);
                _Pragma("unroll") for (int u = 1; u < NW; ++u) t += *reinterpret_cast<const f32x4*>(Pp + u * 1024 + (g * 64 + lane) * 4);
                _Pragma("unroll") for (int j = 0; j < 4; ++j) P[4 * g + j] = t[j];
            }
            return P;
        };
        auto diagonal = [&](const f32x16& P) {  // P[p][p] for this lane's position
            const int l = fresh() & 63;
            float t = 0.f;
            _Pragma("unroll") for (int x = 0; x < 16; ++x) t += hrow(x, l >> 5) == (l & 31) ? P[x] : 0.f;
            return t + __shfl_xor(t, 32, 64);
        };
        for (int kk = 0; kk < s.cnt; ++kk) {
            const ChunkPos cp = walk_step(d, s, rev, kk);
            const int L = cp.L;
            f32x16 O, P;
            float pd = 0.f;
            f32x4 z[4];
            unit_dot(kk);
            __syncthreads();  // (A)
            // the elements that the output is multiplied with, requested before this step's stores: a load waits for the stores before it
            decltype(load4raw(static_cast<const TIO*>(R.aux))) q4[4];
            if (VEC == 2 && R.xdot) {  // (dq and dk only)
                const int l = fresh() & 63, n = min(l & 31, L - 1);
                const size_t row = (cp.tok0 + size_t(rev ? L - 1 - n : n) * cp.ts) * a.vd + vcol + 32 * w + 4 * (l >> 5);
                _Pragma("unroll") for (int g = 0; g < 4; ++g) q4[g] = load4raw(static_cast<const TIO*>(R.aux) + row + 8 * g);
            }
            if constexpr (SUM) {
                __syncthreads();  // (B)
                update(L);
            } else {
                if constexpr (VEC == 1) {
                    P = score_part(K, Q, LQ);
                    {
                        const int l = fresh() & 63;
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) P[x] = hrow(x, l >> 5) == (l & 31) ? P[x] : 0.f;
                    }
                    __syncthreads();  // (B)
                    O = inter(W0, LW);
                    __syncthreads();  // (B2)
                    levels([&](auto lvc, float* cur, float*) {
                        constexpr int lv = decltype(lvc)::value;
                        const f32x16 G = score_part(cur, cur, LW);
                        const int l = fresh() & 63, n = l & 31;
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
                            const int r = hrow(x, l >> 5);
                            if (r < n && (r ^ n) >= lv && (r ^ n) < 2 * lv) P[x] = G[x];
                        }
                        if constexpr (TV == 128 || KD == 256) formed(P);
                        if constexpr (lv == 1) block_store(P);
                        __syncthreads();  // (L)
                    });
                    P = part_sum();
                    pd = diagonal(P);
                    const int l = fresh() & 63;
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) P[x] = hrow(x, l >> 5) == (l & 31) ? 0.f : P[x];
                    __syncthreads();  // (M)
                    const f32x16 X = causal_product<0>(V + 32 * w, LV, P, fresh() & 63, [](int s, int p) { return s < p; });
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) O[x] += X[x];
                    if constexpr (TV == 128 || KD == 256) formed(O);
                } else {
                    if constexpr (RAW) block_store(score_raw());
                    else block_store(score_part(K, Q, LQ));
                    O = inter(Q, LQ);
                    __syncthreads();  // (B)
                    scale_inter(O);
                    P = part_sum();
                    pd = diagonal(P);
                    __syncthreads();  // (B2)
                    levels([&](auto lvc, float* cur, float*) {
                        constexpr int lv = decltype(lvc)::value;
                        f32x16 G;
                        const int l = fresh() & 63, n = l & 31, half = l >> 5;
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
                            const int r = hrow(x, half);
                            G[x] = r < n && (r ^ n) >= lv && (r ^ n) < 2 * lv ? P[x] : 0.f;
                        }
                        const f32x16 X = causal_product<lv>(cur + 32 * w, LW, G, l, [](int r, int p) { return r < p && (r ^ p) >= lv && (r ^ p) < 2 * lv; });
                        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                            const f32x4 e = *reinterpret_cast<const f32x4*>(cur + n * LW + 32 * w + 8 * g + 4 * half);
                            _Pragma("unroll") for (int j = 0; j < 4; ++j) O[4 * g + j] += (n & lv) ? X[4 * g + j] * e[j] : 0.f;
                        }
                        formed(O);
                        __syncthreads();  // (L)
                    });
                }
                update(L);
                unit_keep(kk);
                const int l = fresh() & 63;
                _Pragma("unroll") for (int g = 0; g < 4; ++g) z[g] = *reinterpret_cast<const f32x4*>(V + (l & 31) * LV + 32 * w + 8 * g + 4 * (l >> 5));
            }
            __syncthreads();  // (C)
            if constexpr (!SUM) {
                // The output: the other group's half of the inter product, and the pair (p, p), which stays out of the
                // product with aux: it is the same number in q.dq and in k.dk and cancels in the decay gradient, exactly
                // instead of to rounding.
                const int l = fresh() & 63, n = l & 31, half = l >> 5;
                const int tok = rev ? L - 1 - n : n;           // token of this lane's position (n < L)
                const size_t orow = cp.tok0 + size_t(n < L ? tok : 0) * cp.ts;
                const size_t oel = orow * a.vd + vcol + 32 * w + 4 * half;  // + 8g: four consecutive output features
                _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                    f32x4 o = *reinterpret_cast<const f32x4*>(Pp + w * 1024 + (g * 64 + l) * 4);
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) o[j] += O[4 * g + j];
                    if (VEC == 2 && R.xdot) {
                        const f32x4 q = numbers4(q4[g]);
                        f32x4 y;
                        _Pragma("unroll") for (int j = 0; j < 4; ++j) y[j] = q[j] * o[j];
                        if (n < L) store4(R.xdot + (cp.wtok0 + tok) * a.vd + vcol + 32 * w + 4 * half + 8 * g, y);
                    }
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) o[j] += pd * z[g][j];
                    if (n < L) store4(static_cast<TIO*>(R.out) + oel + 8 * g, o);
                }
            }
        }
    }

    float* e = nullptr;
    if (SUM) e = R.bound + bound_at(R.per, s.slot0, s.unit0, s.wseg + 1) * sz;
    else if (s.empty || s.wseg == s.nsq - 1) e = R.edge_out ? R.edge_out + size_t(s.walk.edge) * sz : nullptr;
    if (e) state_store(S, e, R.trans, a.kd, a.vd, kcol, vcol + 32 * w, fresh() & 63);
}

// States at the segment boundaries of a sequence, in walk order: E_0 = edge_in, E_{s+1} = e^{g_s} E_s + U_s, in place (slot
// s+1 holds U_s on entry).  Elementwise, four elements per thread.
// grid: (d_k d_v / 1024, sequences, directions)
__global__ __launch_bounds__(256) void gk_scan(Dims d, GArgs a) {
    const GRole& R = a.role[blockIdx.z];
    const int q = blockIdx.y, sz = d.dk * d.dv;
    SeqWalk w;
    size_t slot0, unit0;
    if (!d.cu) {
        w = SeqWalk{q, q, 0, 0, 0, d.T};
        slot0 = size_t(q) * a.slots;
        unit0 = size_t(q) * a.units;
    } else {
        const int s = q / d.H;
        w = SeqWalk{q % d.H, q, 0, 0, d.cu[s], d.cu[s + 1]};
        slot0 = size_t(q % d.H) * a.slots + seg_base(d, a.m, s);
        unit0 = size_t(q % d.H) * a.units + d.cstart[s];
    }
    unit0 *= dg_per(d);
    const int nsq = (w.tend - w.tbeg + d.gC * a.m - 1) / (d.gC * a.m);
    const int e = (blockIdx.x * 256 + threadIdx.x) * 4, i = e / d.dv, dkd = d.dkd();
    f32x4 E = {0.f, 0.f, 0.f, 0.f};
    if (R.edge_in) E = load4(R.edge_in + size_t(w.edge) * sz + e);
    // bound_at() as a base and a stride (the rule itself in the loop: 11.8 -> 16.6 us, 28 segments of 32 sequences, d = 64)
    const ptrdiff_t stride = ptrdiff_t(R.per ? R.per : 1) * sz;
    float* b = R.bound + (R.per ? ptrdiff_t(unit0) - 1 : ptrdiff_t(slot0)) * sz + e;
    // A batch of segments costs one memory latency: every load is issued before the first use.  The decays of the scalar
    // kinds are the same for a whole workgroup and come through the scalar cache.
    const double* gp = d.kind == 0 ? nullptr : R.gseg + slot0 * dkd;
    auto chain = [&](auto vec) {
        constexpr int AHEAD = 8;
        for (int s = 0; s + 1 < nsq; s += AHEAD) {
            f32x4 u[AHEAD];
            double gl[AHEAD];
            _Pragma("unroll") for (int x = 0; x < AHEAD; ++x) {
                const int t = min(s + x, nsq - 2);
                u[x] = load4(b + (t + 1) * stride);
                if constexpr (decltype(vec)::value) gl[x] = gp[size_t(t) * dkd + i];
                else gl[x] = gp ? gp[t] : 0.0;
            }
            _Pragma("unroll") for (int x = 0; x < AHEAD; ++x) {
                if (s + x >= nsq - 1) break;
                const float lam = expf(float(gl[x]));
                _Pragma("unroll") for (int c = 0; c < 4; ++c) E[c] = lam * E[c] + u[x][c];
                store4(b + (s + x + 1) * stride, E);
            }
        }
    };
    if (d.kind == 3) chain(std::true_type{});
    else chain(std::false_type{});
}

// Decay gradient of a unit: dg_t = sum_{u >= t in the unit} (q_u.dq_u - k_u.dk_u) + <S_end, dS_end>, S_end / dS_end the
// state and its gradient at the unit's end (vector kind: everything per key feature).  The per-token products come from
// the dq and dk walkers without the pair (t, t), which is the same in both; the last term from the dk walker.
// Scalar kinds: a wave per unit; vector kind: a workgroup.   grid: (ceil(units / 4) or units, heads or sequences)
struct GDgArgs { const float *xq, *xk; const double* z; float *dg, *dg_tok; int units, nslk; };
__global__ __launch_bounds__(256) void gk_dg(Dims d, GDgArgs a) {
    __shared__ double part[256];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), y = blockIdx.y, per = dg_per(d);
    const int x = d.kind == 3 ? blockIdx.x : 4 * blockIdx.x + w;
    if (x >= a.units * per) return;
    int u = x, lo = 0, hi = d.T;
    if (d.cu) {
        const int s = last_seq(d, x, [&](int s) { return d.cstart[s] * per; });
        u = x - d.cstart[s] * per;
        lo = d.cu[s];
        hi = d.cu[s + 1];
    }
    const int tb = lo + u * dg_unit(d), len = min(dg_unit(d), hi - tb);
    if (len <= 0) return;
    const ChunkPos cp = chunk_pos_at(d, y, tb, len, 0);
    const size_t unit = size_t(y) * a.units * per + x;
    if (d.kind != 3) {
        double run = 0.0;
        for (int i = 0; i < d.dk / 32; ++i) run += a.z[unit * (d.dk / 32) + i];
        const size_t plane = size_t(d.BH()) * d.T;
        for (int t0 = len - 1; t0 >= 0; t0 -= 64) {  // 64 tokens at a time, lane l = token t0 - l
            const int t = t0 - lane;
            double v = 0.0;
            if (t >= 0) {
                const size_t row = cp.wtok0 + t;
                for (int sl = 0; sl < a.nslk; ++sl) v += double(a.xq[sl * plane + row]) - double(a.xk[sl * plane + row]);
            }
            for (int off = 1; off < 64; off <<= 1) {
                const double o = __shfl_up(v, off, 64);
                if (lane >= off) v += o;
            }
            v += run;
            if (t >= 0) {
                if (d.kind == 2) a.dg[cp.tok0 + size_t(t) * cp.ts] = float(v);
                else a.dg_tok[cp.wtok0 + t] = float(v);
            }
            run = __shfl(v, 63, 64);
        }
        return;
    }
    // feature i, group gr of the tokens: the group's sum first, then the suffix with the later groups' sums
    const int i = tid % d.dk, ng = 256 / d.dk, gr = tid / d.dk, num = (len + ng - 1) / ng;
    const int first = min(len, gr * num), end = min(len, first + num);
    const float *xq = a.xq + cp.wtok0 * d.dk + i, *xk = a.xk + cp.wtok0 * d.dk + i;
    double sum = 0.0;
    _Pragma("unroll 8") for (int t = first; t < end; ++t) sum += double(xq[size_t(t) * d.dk]) - double(xk[size_t(t) * d.dk]);
    part[gr * d.dk + i] = sum;
    __syncthreads();
    double run = a.z[unit * 2 * d.dk + i] + a.z[(unit * 2 + 1) * d.dk + i];
    for (int h = gr + 1; h < ng; ++h) run += part[h * d.dk + i];
    _Pragma("unroll 8") for (int t = end - 1; t >= first; --t) {
        run += double(xq[size_t(t) * d.dk]) - double(xk[size_t(t) * d.dk]);
        a.dg[(cp.tok0 + size_t(t) * cp.ts) * d.dk + i] = float(run);
    }
}

// dg[h] = sum_{b,t} dg_tok[b,h,t], fixed summation order (grid: H)
__global__ __launch_bounds__(1024) void gk_head_reduce(Dims d, const float* __restrict__ dg_tok, float* __restrict__ dg) {
    __shared__ double part[1024];
    const int h = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    for (int b = 0; b < d.B; ++b) {
        const float* x = dg_tok + (size_t(b) * d.H + h) * d.T;
        _Pragma("unroll 4") for (int t = tid; t < d.T; t += 1024) s += double(x[t]);
    }
    part[tid] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) part[tid] += part[tid + w];
        __syncthreads();
    }
    if (tid == 0) dg[h] = float(part[0]);
}

// packed input: cstart[s] = sum over earlier sequences of max(least, ceil(len / C))  (one thread; n_seq is small)
__global__ void k_chunk_starts(Dims d, int* __restrict__ cstart, int least) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int c = 0;
    cstart[0] = 0;
    for (int s = 0; s < d.nseq; ++s) {
        c += max(least, (d.cu[s + 1] - d.cu[s] + d.C - 1) / d.C);
        cstart[s + 1] = c;
    }
}

// ---- host side --------------------------------------------------------------------------------------------------

// Segment plan: m units of gC tokens per segment.  Enough workgroups that the launch fills the chip with what fits on a
// compute unit (two of the 128-wide walkers, four of the 64-wide ones), and no more boundary states than one per chunk of
// the caller's chunk size, which is what lsm_chunk_fwd_workspace_bytes() has always reported.
// Half as many, as many and twice as many workgroups, us a call: 32 sequences of 1777, d = 64, forward 52 / 47 / 47; 64 of 1024,
// d = 64, fp32, 62 / 52 / 52; 32 of 2048, d_k = 64, d_v = 128, 68 / 54 / 68, vector kind with backward 544 / 439 / 479; 64 of 1000,
// d = 128, fp32, 111 / 94 / 117.  Half is the better one for many short sequences (256 of 256, d = 128, fp32: 66 / 95 / 115).
// (Of the scalar kinds' fp32 walkers with 128- and 256-wide keys two and one fit; the plan counts four for every 64-wide value.)
struct GPlan { int m, nseg, units; };  // nseg: segments (and boundary slots), units: of gC tokens, per sequence or per head
int slices(int width, bool narrow) { return narrow ? width / 64 : (width + 127) / 128; }
GPlan gplan(const Dims& d) {
    const int units = (d.T + d.gC - 1) / d.gC, nsl = slices(d.dv, false), target = d.dv == 64 ? 1024 : 512;
    GPlan p{};
    if (!d.nseq) {
        const int seqs = d.BH() * nsl;
        int nseg = (target + seqs - 1) / seqs;
        nseg = nseg > units ? units : nseg;
        p.m = (units + nseg - 1) / nseg;
        p.nseg = (units + p.m - 1) / p.m;
        p.units = units;
        return p;
    }
    const long long n = (long long)units + d.nseq, work = n * d.H * nsl;
    p.m = int((work + target - 1) / target);
    auto count = [&](int m) { return m == 1 ? int(n) : int(n / m) + d.nseq + 1; };
    while (count(p.m) > n) ++p.m;  // n: the chunks the workspace figure allows for
    p.nseg = count(p.m);
    p.units = int(n);
    return p;
}

struct GWs { float *bound_f, *bound_r, *xq, *xk, *dg_tok; double *gseg_f, *gseg_r, *z; size_t bytes; };
GWs carve(const Dims& d, void* ws, bool bwd) {
    char* p = static_cast<char*>(ws);
    size_t off = 0;
    GWs w{};
    const GPlan gp = gplan(d);
    auto take = [&](size_t bytes) { char* r = p + off; off += align256(bytes); return r; };
    const size_t rows = d.nseq ? d.H : d.BH(), slots = gp.nseg > 1 ? gp.nseg * rows : 0;
    // backward: a state per decay-gradient unit, the segments' entry states among them
    const size_t units = bwd && d.kind != 0 ? size_t(gp.units) * dg_per(d) * rows : 0;
    const size_t st = size_t(d.dk) * d.dv * 4, ng = d.kind != 0 ? slots * d.dkd() * 8 : 0;
    w.bound_f = reinterpret_cast<float*>(take((slots > units ? slots : units) * st));
    w.gseg_f = reinterpret_cast<double*>(take(ng));
    if (bwd) {
        w.bound_r = reinterpret_cast<float*>(take(slots * st));
        w.gseg_r = reinterpret_cast<double*>(take(ng));
        const size_t tok = size_t(d.BH()) * d.T;
        const size_t nx = d.kind == 0 ? 0 : tok * (d.kind == 3 ? d.dk : slices(d.dk, false)) * 4;
        w.xq = reinterpret_cast<float*>(take(nx));
        w.xk = reinterpret_cast<float*>(take(nx));
        w.z = reinterpret_cast<double*>(take(units * (d.kind == 3 ? 2 * d.dk : d.dk / 32) * 8));
        if (d.kind == 1) w.dg_tok = reinterpret_cast<float*>(take(tok * 4));
    }
    w.bytes = off;
    return w;
}
// The size the queries report: at least one fp32 state per chunk of the caller's chunk size (twice for the backward call)
// and one running log-decay per token, as callers have always been told (the forward figure also decides what fits the
// built-in scratch of lsm_chunk_fwd_noalloc).  The forward kernels use less; the backward ones a state per decay-gradient unit
// and per segment, and less than the figure too (but for packed batches with more empty sequences than chunks).
size_t reported(const Dims& d, bool bwd) {
    const size_t tok = size_t(d.BH()) * d.T, st = align256(size_t(d.BH()) * d.N * d.dk * d.dv * 4);
    size_t n = (d.kind != 0 ? align256(tok * d.dkd() * 8) : 0) + st;
    if (bwd) n += st + (d.kind != 0 ? 2 * align256(tok * d.dk * 4) : 0) + (d.kind == 1 ? align256(tok * 4) : 0);
    return n;
}

// dynamic LDS limit of a kernel, raised once per kernel and device
hipError_t allow_lds(const void* fn, int bytes) {
    struct Seen { const void* fn; uint64_t devices; };
    static std::mutex mu;
    static std::vector<Seen> seen;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = uint64_t(1) << (dev & 63);
    std::lock_guard<std::mutex> lk(mu);
    for (Seen& x : seen)
        if (x.fn == fn) {
            if (x.devices & bit) return hipSuccess;
            if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)) == hipSuccess) x.devices |= bit;
            return e;
        }
    if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)) == hipSuccess) seen.push_back(Seen{fn, bit});
    return e;
}

static_assert(GLdsS<float, 64, 64, 0, false>::bytes <= 40 * 1024, "four workgroups to a compute unit: gplan");
template <typename TIO, int KD, int TV, int VEC, int HW, bool SUM>
hipError_t launch_walk_as(const Dims& d, GArgs a, int nroles, dim3 grid, hipStream_t st, int kid) {
    using Lds = std::conditional_t<VEC == 0, GLdsS<TIO, KD, TV, HW, SUM>, GLds<TIO, KD, TV, VEC, SUM>>;
    static_assert(Lds::bytes <= 160 * 1024, "LDS");
    void (*kernel)(Dims, GArgs);
    if constexpr (VEC == 0) kernel = gk_walk<TIO, KD, TV, HW, SUM>;
    else kernel = gk_walk_vec<TIO, KD, TV, VEC, SUM>;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(kernel), Lds::bytes);
    if (e != hipSuccess) return e;
    a.nsl = a.vd / TV;
    grid.z = nroles * a.nsl;
    ProfScope ps(kid, st);
    hipLaunchKernelGGL(kernel, grid, dim3(VEC == 0 ? 2 * TV + 64 * HW : 4 * TV), Lds::bytes, st, d, a);
    return hipGetLastError();
}
template <typename TIO, int KD, int TV, int VEC, bool SUM>
hipError_t launch_walk(const Dims& d, const GArgs& a, int nroles, dim3 grid, hipStream_t st, int kid) {
    // Two more waves for the rows, the tables and the scores where every workgroup has a compute unit to itself: a step is then
    // one wave's chain of instructions.  us a call without and with them: 2 sequences of 256, fp32, d = 64 26.8 / 23.6, 128-wide keys
    // 39.9 / 33.9, 256-wide 57.3 / 49.0, their training steps 112 / 99 and 148 / 131; 8 of 2000, fp32 52 / 46 and 71 / 60, bf16 44 / 41 and
    // 56 / 51.  With 3.5 workgroups to a unit (32 of 1777, bf16, d = 64) 42.4 / 52.0.
    if constexpr (VEC == 0 && TV == 64)
        if (grid.x * grid.y * unsigned(nroles * (a.vd / TV)) <= 256) return launch_walk_as<TIO, KD, TV, VEC, 2, SUM>(d, a, nroles, grid, st, kid);
    return launch_walk_as<TIO, KD, TV, VEC, 0, SUM>(d, a, nroles, grid, st, kid);
}
// Key-role width kd keeps its whole state column block in one wave's registers; value-role widths of 128 and 256 go in
// slices of 128 (fewer repeats of the scores), except the vector kind's with 256-wide keys (LDS, registers).
template <typename TIO, int VEC, bool SUM>
hipError_t walk_dims(const Dims& d, const GArgs& a, int nroles, dim3 grid, hipStream_t st, int kid) {
    const bool narrow = a.vd == 64;
    if (a.kd == 64) return narrow ? launch_walk<TIO, 64, 64, VEC, SUM>(d, a, nroles, grid, st, kid) : launch_walk<TIO, 64, 128, VEC, SUM>(d, a, nroles, grid, st, kid);
    if (a.kd == 128) return narrow ? launch_walk<TIO, 128, 64, VEC, SUM>(d, a, nroles, grid, st, kid) : launch_walk<TIO, 128, 128, VEC, SUM>(d, a, nroles, grid, st, kid);
    if constexpr (VEC != 0) return launch_walk<TIO, 256, 64, VEC, SUM>(d, a, nroles, grid, st, kid);
    else return narrow ? launch_walk<TIO, 256, 64, VEC, SUM>(d, a, nroles, grid, st, kid) : launch_walk<TIO, 256, 128, VEC, SUM>(d, a, nroles, grid, st, kid);
}
template <typename TIO>
hipError_t walks(const Dims& d, const GArgs& a, int nroles, dim3 grid, hipStream_t st) {
    // the decayed features are d_k's: on the key side of o and dv, on the value side (the transposed state) of dq and dk
    if (d.kind != 3) return walk_dims<TIO, 0, false>(d, a, nroles, grid, st, a.role[0].trans ? KID_GEN_GRAD : KID_GEN_OUTPUT);
    return a.role[0].trans ? walk_dims<TIO, 2, false>(d, a, nroles, grid, st, KID_GEN_GRAD)
                           : walk_dims<TIO, 1, false>(d, a, nroles, grid, st, KID_GEN_OUTPUT);
}
template <typename TIO>
hipError_t bounds(const Dims& d, const GArgs& a, int ndir, dim3 grid, hipStream_t st) {
    const hipError_t e = d.kind != 3 ? walk_dims<TIO, 0, true>(d, a, ndir, grid, st, KID_GEN_STATE) : walk_dims<TIO, 1, true>(d, a, ndir, grid, st, KID_GEN_STATE);
    if (e != hipSuccess) return e;
    ProfScope ps(KID_GEN_SCAN, st);
    hipLaunchKernelGGL(gk_scan, dim3(d.dk * d.dv / 1024, d.seqs(), ndir), dim3(256), 0, st, d, a);
    return hipGetLastError();
}

template <typename TIO>
hipError_t fwd_t(const Dims& d, const FwdArgs& f) {
    const GWs w = carve(d, f.ws, false);
    const GPlan gp = gplan(d);
    const dim3 grid(gp.nseg, d.nseq ? d.H : d.BH());
    GArgs a{};
    a.g = f.g; a.kd = d.dk; a.vd = d.dv; a.m = gp.m; a.slots = gp.nseg; a.units = gp.units;
    a.role[0] = GRole{f.q, f.k, f.v, nullptr, f.o, nullptr, f.m0, f.mT, w.bound_f, w.gseg_f, 0, 0};
    if (gp.nseg > 1) {
        const hipError_t e = bounds<TIO>(d, a, 1, grid, f.stream);
        if (e != hipSuccess) return e;
    }
    return walks<TIO>(d, a, 1, grid, f.stream);
}

template <typename TIO>
hipError_t bwd_t(const Dims& d, const BwdArgs& b) {
    const GWs w = carve(d, b.ws, true);
    const GPlan gp = gplan(d);
    const dim3 grid(gp.nseg, d.nseq ? d.H : d.BH());
    hipError_t e;
    const bool want_dg = b.dg != nullptr;
    const int per = want_dg ? gp.m * dg_per(d) : 0;
    GArgs a{};
    a.g = b.g; a.kd = d.dk; a.vd = d.dv; a.m = gp.m; a.slots = gp.nseg; a.units = gp.units;
    a.role[0] = GRole{nullptr, b.k, b.v, nullptr, nullptr, nullptr, b.m0, nullptr, w.bound_f, w.gseg_f, 0, 0, per};
    a.role[1] = GRole{nullptr, b.q, b.d_o, nullptr, nullptr, nullptr, b.d_mT, nullptr, w.bound_r, w.gseg_r, 1, 0};
    if (gp.nseg > 1 && (e = bounds<TIO>(d, a, 2, grid, b.stream)) != hipSuccess) return e;
    float *xq = want_dg ? w.xq : nullptr, *xk = want_dg ? w.xk : nullptr;
    const GRole dq{b.d_o, b.v, b.k, b.q, b.dq, xq, b.m0, nullptr, w.bound_f, nullptr, 0, 1, per, want_dg ? (b.d_mT ? 2 : 1) : 0};
    const GRole dk{b.v, b.d_o, b.q, b.k, b.dk, xk, b.d_mT, nullptr, w.bound_r, nullptr, 1, 1, 0, 0, want_dg ? w.bound_f : nullptr, w.z};
    const GRole dv{b.k, b.q, b.d_o, nullptr, b.dv, nullptr, b.d_mT, b.d_m0, w.bound_r, nullptr, 1, 0};
    auto walk = [&](std::initializer_list<GRole> roles) {  // roles of one launch: the same widths
        const bool grad = roles.begin()->trans != 0;
        a.kd = grad ? d.dv : d.dk; a.vd = grad ? d.dk : d.dv;
        std::copy(roles.begin(), roles.end(), a.role);
        return walks<TIO>(d, a, int(roles.size()), grid, b.stream);
    };
    const bool one = d.dk == d.dv && d.kind != 3;  // one launch may hold dv as well
    if (want_dg) {  // the dk walker reads what the dq walker leaves
        if ((e = one ? walk({dq, dv}) : walk({dq})) != hipSuccess || (e = walk({dk})) != hipSuccess) return e;
    } else if ((e = one ? walk({dq, dk, dv}) : walk({dq, dk})) != hipSuccess) {
        return e;
    }
    if (!one && (e = walk({dv})) != hipSuccess) return e;
    if (want_dg) {
        const GDgArgs ga{w.xq, w.xk, w.z, b.dg, w.dg_tok, gp.units, slices(d.dk, false)};
        const int units = gp.units * dg_per(d);
        {
            ProfScope ps(KID_GEN_DG, b.stream);
            hipLaunchKernelGGL(gk_dg, dim3(d.kind == 3 ? units : (units + 3) / 4, grid.y), dim3(256), 0, b.stream, d, ga);
        }
        if (d.kind == 1) {
            ProfScope ps(KID_HEAD_REDUCE, b.stream);
            hipLaunchKernelGGL(gk_head_reduce, dim3(d.H), dim3(1024), 0, b.stream, d, w.dg_tok, b.dg);
        }
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_chunk_starts(const Dims& d, int* cstart, hipStream_t stream) {
    hipLaunchKernelGGL(k_chunk_starts, dim3(1), dim3(64), 0, stream, d, cstart, 0);
    return hipGetLastError();
}
// the walkers' table: in units of gC tokens, an empty sequence holding one (its workgroup passes the state through)
hipError_t launch_generic_starts(const Dims& d, int* cstart, hipStream_t stream) {
    Dims u = d;
    u.C = d.gC;
    hipLaunchKernelGGL(k_chunk_starts, dim3(1), dim3(64), 0, stream, u, cstart, 1);
    return hipGetLastError();
}

size_t generic_fwd_workspace(const Dims& d) {
    const size_t need = carve(d, nullptr, false).bytes, rep = reported(d, false);
    return need > rep ? need : rep;
}
size_t generic_bwd_workspace(const Dims& d) {
    const size_t need = carve(d, nullptr, true).bytes, rep = reported(d, true);
    return need > rep ? need : rep;
}

hipError_t generic_fwd(const Dims& d, const FwdArgs& a) {
    return d.bf16 ? fwd_t<uint16_t>(d, a) : fwd_t<float>(d, a);
}
hipError_t generic_bwd(const Dims& d, const BwdArgs& a) {
    return d.bf16 ? bwd_t<uint16_t>(d, a) : bwd_t<float>(d, a);
}

}  // namespace lsm
