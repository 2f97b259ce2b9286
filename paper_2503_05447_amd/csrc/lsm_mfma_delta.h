// Delta-rule rows of the paper's Table 1 (DeltaNet, Gated DeltaNet), chunkwise: bf16 operands, fp32
// accumulation, chunk = 64, d_k = d_v = 128.  Included by lsm_mfma.hip after lsm_mfma_walk.h.
//
// Both rows are  M_t = alpha_t (I - beta_t k_t^T k_t) M_{t-1} + b_t k_t^T v_t ,  o_t = q_t M_t  (DeltaNet:
// alpha = 1, beta = the row's a_t; Gated DeltaNet: alpha = the row's a_t, beta = 1).  With the pseudo-value
//     u_t = b_t v_t - alpha_t beta_t k_t M_{t-1}
// the update reads M_t = alpha_t M_{t-1} + k_t^T u_t: the per-token scalar-decay recurrence of Eq. 5 with u in
// the place of v, which the chunk walker already evaluates.  Inside a chunk that starts from the state S, with
// Gamma_t = prod_{s <= t} alpha_s, the pseudo-values solve the unit lower-triangular system
//     (I + L) U = R ,  R = diag(b) V - diag(beta Gamma) K S ,   L_tr = beta_t (Gamma_t / Gamma_r) (k_t . k_r) ,  r < t
// (the chunkwise form published for the delta rule; the paper itself gives no algorithm for these rows).
//   mk_delta_prep  (one workgroup per chunk, all chunks in parallel): L from K K^T on the matrix cores, T = (I + L)^-1 by
//                  forward substitution in fp32 inside 32 x 32 diagonal blocks and a block product below them.
//   mk_delta_walk8 (one workgroup per sequence or segment): the forward chunk walker with two more products per chunk,
//                  K S from the state in the accumulators and U = T R; U then plays the values' part in the
//                  intra-chunk product and in the state update.
// T is all that is handed from one to the other, without its diagonal: U = R + (T - I) R, in reverse W = dU + (T - I)^T dU, so that
// R and dU, split for the products, are not rounded where they stand for themselves.  (2-norm errors with T whole, 16 x 16
// sequences of 2048: d beta 8.8e-6, d b 3.5e-6, final state 3.6e-6; so 8.2e-6, 2.5e-6, 2.7e-6.)  (T diag(b) V in fp32 and T diag(beta Gamma) K in bf16, formed by the first kernel,
// make the walk's chain one product shorter and cost 1.3 KB of traffic a token and the rounding of the latter: 16 x 16
// sequences of 2048, keeping U, 209 + 251 us; this 74 + 198.  Final state without a decay, 2-norm error 4.6e-4 -> 4.0e-6.)
// Every value column of the state evolves on its own (the erase term acts on the key side only), so a wave
// keeps its 128 x 32 slice of S and its 32 columns of R and U to itself, in registers throughout: lane = value column,
// registers = the index that the next product contracts.
// Segments.  The state a segment of chunks ends with is an affine function of the state it starts from, S' = A S + B,
// with a dense d_k x d_k factor A (the product of the chunks' erase-and-decay factors), not a decayed sum.  Because
// the value columns evolve independently, A is what the same walk makes of the identity when the values are zero,
// and B what it makes of a zero state: with fewer sequences than compute units, a summary pass runs the state part
// of the walker twice per segment (MODE 1: B, MODE 2: A), mk_delta_combine chains E' = A E + B over the segments of
// each sequence on the matrix cores, and the walker proper then runs all segments in parallel.
#pragma once

constexpr int LDD = 36;      // floats per row of a 32 x 32 diagonal block of L
constexpr int LDT = 40;      // elements per row of a 32 x 32 bf16 tile
// T^T (rows r, columns t) of a chunk in memory, bf16 head and remainder: the rows r < 32 of either plane (64 columns), then the
// rows r >= 32 (columns 32 .. 63; the others are zero and not kept); zeros in the place of the ones on the diagonal
constexpr int kDeltaT = 2 * 32 * 64 + 2 * 32 * 32;
// its 16-byte pieces in that order: place of piece p in a pair of tiles [2][64][LDP]
__device__ __forceinline__ int delta_t_place(int p) {
    const int q = p - 512;
    return p < 512 ? ((p >> 8) * C + ((p >> 3) & 31)) * LDP + 8 * (p & 7) : ((q >> 7) * C + 32 + ((q >> 2) & 31)) * LDP + 32 + 8 * (q & 3);
}
// LDS of mk_delta_prep (four workgroups per compute unit): K tile, later L: diagonal blocks (fp32; later R^T head, remainder),
// L_10 head, remainder | T^T head, remainder (64 x LDP) | log Gamma, beta
constexpr int kDeltaPrepLds = C * LD * 2 + 2 * C * LDP * 2 + 2 * C * 4;
static_assert(2 * 32 * LDD * 4 + 2 * 32 * LDT * 2 <= C * LD * 2 && 2 * 32 * LDD * 4 >= 2 * 32 * LDT * 2, "tenants fit");

struct DeltaPrepArgs {
    const uint16_t* k;
    const float *log_alpha, *beta;  // per token ([B,H,T], or [B,T,H] for the token-major layout); NULL = 1
    uint16_t* tt;                   // [BH*N][kDeltaT]
};

// a token-contraction operand like frag_tr whose k order follows a D-layout block (frag_perm's): slot e of lane (n, half) is row
// row0 + 8 (e / 4) + 4 half + e % 4 of column col0 + n
__device__ __forceinline__ bf16x8 frag_tr_perm(const uint16_t* tile, int ld, int row0, int col0, int lane) {
    const int r = lane & 15, nblk = (lane >> 4) & 1, half = lane >> 5;
    const uint16_t* p = tile + (row0 + 4 * half + (r >> 2)) * ld + col0 + 16 * nblk + 4 * (r & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)));
    const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 8 * ld)));
    return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
}
// weights of the rows of registers 8p .. 8p+7 of a D-layout block at row0 - 16p
__device__ __forceinline__ void row_weights(const float* tab, int row0, int half, float (&w)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(tab + row0 + 4 * half), b = *reinterpret_cast<const float4*>(tab + row0 + 8 + 4 * half);
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w; w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
}

// 32 consecutive fp32 values -> one 32-element bf16 row, head and remainder
__device__ __forceinline__ void delta_row_split(uint16_t* hi, uint16_t* lo, const float (&x)[32]) {
    _Pragma("unroll") for (int i = 0; i < 4; ++i) {
        u32x4 h, l;
        _Pragma("unroll") for (int p = 0; p < 4; ++p) {
            const float x0 = x[8 * i + 2 * p], x1 = x[8 * i + 2 * p + 1];
            h[p] = pack2(x0, x1);
            l[p] = pack2(x0 - bf16_lo(h[p]), x1 - bf16_hi(h[p]));
        }
        *reinterpret_cast<u32x4*>(hi + 8 * i) = h;
        *reinterpret_cast<u32x4*>(lo + 8 * i) = l;
    }
}

// grid: (N, BH).  T = (I + L)^-1 in two levels: the two 32 x 32 diagonal blocks by forward substitution in fp32
// (one wave, lane = block and column), the block below the diagonal as T_10 = -T_11 L_10 T_00 on the matrix cores
// with every factor as bf16 head + remainder.  T is kept transposed, so every lane writes whole 16-byte row pieces.
// Bound: one wave's chain of the substitution (2.4 us of 5); four workgroups to a compute unit run beside each other.
template <bool DEC>
__global__ __launch_bounds__(kThreads, 4) void mk_delta_prep(Dims d, DeltaPrepArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* Kt = reinterpret_cast<uint16_t*>(smem);
    float* Ld = reinterpret_cast<float*>(smem);                            // [2][32][LDD]: L_00, L_11
    uint16_t* RTh = reinterpret_cast<uint16_t*>(smem);                     // over L_00, L_11 once they are spent
    uint16_t* RTl = RTh + 32 * LDT;
    uint16_t* L10h = reinterpret_cast<uint16_t*>(smem + 2 * 32 * LDD * 4); // L_10 [t'][r]
    uint16_t* L10l = L10h + 32 * LDT;
    uint16_t* Th = Kt + C * LD;                                            // T^T [r][t]
    uint16_t* Tl = Th + C * LDP;
    float* lg = reinterpret_cast<float*>(Tl + C * LDP);                    // log Gamma_t
    float* be = lg + C;

    const int c = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, half = lane >> 5;
    const ChunkPos cp = chunk_pos(d, c, bh);
    const int L = cp.L;
    if (L <= 0) return;
    TileRegs rk;
    tile_gload(rk, a.k, cp.tok0, cp.ts, L, tid);
    if (wave == 0) {
        const size_t ptok = cp.tok0 + size_t(min(lane, L - 1)) * cp.ts;
        float x = (DEC && lane < L) ? a.log_alpha[ptok] : 0.f;
        const float bet = a.beta ? a.beta[ptok] : 1.f;
        for (int off = 1; off < 64; off <<= 1) {
            const float y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        lg[lane] = x;
        be[lane] = lane < L ? bet : 0.f;  // rows beyond the ragged end: no erase
    }
    tile_commit(Kt, rk, L, tid);
    __syncthreads();
    // ---- L[t][r] = beta_t e^{lg_t - lg_r} (k_t . k_r) for r < t, else 0: blocks (r, t) = (0,0), (0,1), (1,1)
    f32x16 G;
    const int rb = wave == 2 ? 1 : 0, tb = wave ? 1 : 0;
    if (wave < 3) {
        G = score_block2(Kt, 32 * rb, Kt, 32 * tb, n, half);  // D[m = r][n = t]
        const int t = 32 * tb + n;
        const float bt = be[t], lt = lg[t];
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            const float4 lr = *reinterpret_cast<const float4*>(lg + 32 * rb + 8 * g + 4 * half);
            const float lrv[4] = {lr.x, lr.y, lr.z, lr.w};
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {
                const int r = 32 * rb + 8 * g + 4 * half + j;
                G[4 * g + j] = r < t ? bt * (DEC ? __expf(lt - lrv[j]) : 1.f) * G[4 * g + j] : 0.f;
            }
        }
    }
    __syncthreads();  // the K tile is spent
    if (wave < 3) {
        if (rb == tb) {  // diagonal block, fp32 [t'][r']
            float* dst = Ld + rb * 32 * LDD + n * LDD;
            _Pragma("unroll") for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(dst + 8 * g + 4 * half) = float4{G[4 * g], G[4 * g + 1], G[4 * g + 2], G[4 * g + 3]};
        } else {         // L_10 [t'][r], bf16 head + remainder
            store_block_t_split(L10h, L10l, LDT, n, 0, half, G);
        }
    }
    __syncthreads();
    if (wave == 0) {
        // ---- diagonal blocks: X[t'] = [t' == c] - sum_{r' < t'} L_bb[t'][r'] X[r'], lane = (block, column c)
        const int blk = half, cc = n;
        const float* Lb = Ld + blk * 32 * LDD;
        float X[32];
        _Pragma("unroll") for (int t = 0; t < 32; ++t) X[t] = 0.f;
        _Pragma("unroll") for (int t = 0; t < 32; ++t) {
            float acc[4] = {cc == t ? 1.f : 0.f, 0.f, 0.f, 0.f};
            _Pragma("unroll") for (int q4 = 0; q4 < (t + 3) / 4; ++q4) {
                const float4 l = *reinterpret_cast<const float4*>(Lb + t * LDD + 4 * q4);
                acc[0] -= l.x * X[4 * q4];
                acc[1] -= l.y * X[4 * q4 + 1];
                acc[2] -= l.z * X[4 * q4 + 2];
                acc[3] -= l.w * X[4 * q4 + 3];
            }
            X[t] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        }
        delta_row_split(Th + lane * LDP + 32 * blk, Tl + lane * LDP + 32 * blk, X);
        __builtin_amdgcn_wave_barrier();  // LDS serves one wave's accesses in order: what follows reads what was just written
        // ---- R[r][t] = sum_t' L_10[t'][r] T_11[t][t'], kept as R^T [t][r]
        f32x16 R = {0};
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 ah = frag_tr(L10h, LDT, 16 * ks, 0, lane), al = frag_tr(L10l, LDT, 16 * ks, 0, lane);
            const bf16x8 bh_ = frag_tr(Th, LDP, 32 + 16 * ks, 32, lane), bl = frag_tr(Tl, LDP, 32 + 16 * ks, 32, lane);
            R = mfma(ah, bh_, R);
            R = mfma(ah, bl, R);
            R = mfma(al, bh_, R);
        }
        __builtin_amdgcn_wave_barrier();
        store_block_t_split(RTh, RTl, LDT, n, 0, half, R);  // over the diagonal blocks of L, which are spent
        __builtin_amdgcn_wave_barrier();
        // ---- T_10[t][c] = -sum_r R^T[t][r] T_00[r][c]
        f32x16 T10 = {0};
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 ah = frag(RTh, LDT, n, 16 * ks + 8 * half), al = frag(RTl, LDT, n, 16 * ks + 8 * half);
            const bf16x8 bh_ = frag(Th, LDP, n, 16 * ks + 8 * half), bl = frag(Tl, LDP, n, 16 * ks + 8 * half);
            T10 = mfma(ah, bh_, T10);
            T10 = mfma(ah, bl, T10);
            T10 = mfma(al, bh_, T10);
        }
        _Pragma("unroll") for (int x = 0; x < 16; ++x) T10[x] = -T10[x];
        store_block_t_split(Th, Tl, LDP, n, 32, half, T10);  // rows c, columns 32 + t
        Th[lane * LDP + lane] = 0;  // (after this wave's last read of T; the remainder of a 1 is zero)
    }
    __syncthreads();  // T - I is complete
    _Pragma("unroll") for (int it = 0; it < 3; ++it) {
        const int p = tid + kThreads * it;
        *reinterpret_cast<u32x4*>(a.tt + cp.slot * kDeltaT + 8 * p) = *reinterpret_cast<const u32x4*>(Th + delta_t_place(p));
    }
}

// ---- the walker
struct DeltaWalkArgs {
    const uint16_t *q, *k, *v;
    const uint16_t* tt;     // [BH*N][kDeltaT]
    const float *log_alpha, *beta, *bw;  // per token, NULL = 1
    uint16_t* out;
    const float* edge_in;   // M_0 [i][v] per sequence or NULL
    float* edge_out;        // M_T or NULL
    uint16_t *usave, *usave_l;  // NULL, or the pseudo-values (bf16 head, remainder) in the layout of v, for the backward pass
    // segments (nseg > 1): m chunks each; the walker enters segment s with bound[seq][s]; the summary modes leave their
    // end state in sum[seq][s] ([i][v] fp32, 128 x 128 each)
    int m, nseg;
    const float* bound;
    float* sum;
    // the gradient walker's entry states, where its segments are not this walk's (NULL: they are): the state before every em-th
    // chunk of a sequence, slots as bound_slot() numbers them for en segments a sequence
    float* entries;
    int em, en;
};

// The walk (MODE 0), and the summaries of a segment for the cut into segments: the state part of the walk alone, from a
// zero state (MODE 1: the segment's own contribution B) or from the identity with zero values (MODE 2: its transfer
// matrix A).  grid: (segments, seqs).  Eight waves, two per SIMD, split by function:
//   waves 0..3 carry the state (wave w: value columns [32w, 32w+32)): both inter products, R and U, the intra
//              part of the output and the state update - the chain that every chunk has to go through in order;
//   waves 4..7 do everything that does not need the state: all tile traffic (global -> registers -> LDS one chunk ahead,
//              output and pseudo-values -> global), the tables, the three score blocks.
// A chunk has two phases.  In the first the carrier waves read Q, K, V and T (inter products, R, U) while the others compute
// the scores and store the previous chunk's results; in the second the carrier waves read only the scores and K (intra
// part, state update), so the others overwrite Q, V, T and the K tile of the chunk before with the next chunk's rows and rebuild the
// tables (K and the tables in two sets, used in turn) meanwhile: two barriers a chunk.
// The pseudo-values are kept as bf16 head + remainder: a single rounding of u_t would show in o_t at the size of
// an output ulp wherever one token dominates the read-out (strong decay), which the diagonal kinds never pay
// because their values are inputs.  R is split the same way, products of two remainders are left out.
// LDS: Q | K (two sets) | V | output stage | U head stage | U remainder stage (64 x LD bf16 each) | T^T head | remainder |
// scores head | scores remainder (64 x LDP) | two sets of (bs, wo, -beta Gamma, b)
constexpr int kDeltaTab = 4 * C + 4;
constexpr int kDeltaWalk8Lds = (7 * C * LD + 4 * C * LDP) * 2 + 2 * kDeltaTab * 4;
static_assert(kDeltaWalk8Lds <= 160 * 1024, "one workgroup's LDS");

template <bool DEC, int MODE>
__global__ __launch_bounds__(512, 1) void mk_delta_walk8(Dims d, DeltaWalkArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* Q = reinterpret_cast<uint16_t*>(smem);
    uint16_t* K2 = Q + C * LD;   // [2]
    uint16_t* V = K2 + 2 * C * LD;
    uint16_t* stage = V + C * LD;
    uint16_t* Us = stage + C * LD;
    uint16_t* Usl = Us + C * LD;
    uint16_t* Th = Usl + C * LD;
    uint16_t* Tl = Th + C * LDP;
    uint16_t* Ph = Tl + C * LDP;
    uint16_t* Pl = Ph + C * LDP;
    float* tab = reinterpret_cast<float*>(Pl + C * LDP);  // [2][kDeltaTab]: bs (65), wo, ne, bb (64) of the chunks of either parity

    // the wave index as a scalar: the branch between the two groups is a scalar branch
    const int seg = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave8 & 3;
    int lane = tid & 63, n = lane & 31, half = lane >> 5;
    // (as in mk_walk_grad: a phase's lane-dependent LDS addresses are formed in the phase, not kept across the loop)
    auto fresh = [&]() {
        asm volatile("" : "+v"(lane));
        n = lane & 31;
        half = lane >> 5;
    };
    const int t256 = tid & 255;
    const bool carrier = wave8 < 4;
    const SeqWalk walk = seq_walk(d, seq);
    const int nsq = max(1, (walk.n + a.m - 1) / a.m);  // segments of this sequence
    const int kbeg = seg * a.m, kend = min(walk.n, kbeg + a.m), cnt = max(kend - kbeg, 0);
    if (MODE != 0) {
        // only segments whose end state another one starts from (backward in time the last one's factor is wanted too)
        if (nsq == 1 || cnt <= 0 || (seg == nsq - 1 && !(MODE == 2 && a.usave))) return;
    } else if (seg >= nsq) {
        return;
    }

    if (carrier) {
        f32x16 S[4];
        _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = f32x16{0};
        if (MODE == 0) {
            const float* ein = a.nseg > 1 ? a.bound + (size_t(seq) * a.nseg + seg) * D * D
                                          : (a.edge_in ? a.edge_in + size_t(seq) * D * D : nullptr);
            if (ein) walk_state_load(S, ein, false, wave, n, half);
        } else if (MODE == 2) {
            _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
                _Pragma("unroll") for (int x = 0; x < 16; ++x)
                    S[ib][x] = (32 * ib + 8 * (x >> 2) + 4 * half + (x & 3) == 32 * wave + n) ? 1.f : 0.f;
        }
        for (int kk = 0; kk < cnt; ++kk) {
            const uint16_t* K = K2 + (kk & 1) * C * LD;
            const float* bs = tab + (kk & 1) * kDeltaTab;
            const float *wo = bs + C + 4, *ne = wo + C, *bb = ne + C;
            if (MODE == 0 && a.entries) {
                const int k = kbeg + kk;
                if (k > 0 && k % a.em == 0)
                    walk_state_store(S, a.entries + (bound_slot(d, walk, a.em, a.en) + k / a.em) * D * D, false, wave, n, half);
            }
            __syncthreads();  // (A) the tiles and the tables of this chunk are in LDS
            fresh();
            // both inter products with one conversion of the state blocks: R[t][v] = sum_i k_t[i] S[i][v], O^T[v][j] = sum_i S[i][v] q_j[i]
            f32x16 R[2] = {{0}, {0}}, O[2] = {{0}, {0}};
            _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
                _Pragma("unroll") for (int p = 0; p < 2; ++p) {
                    u32x4 hi, lo;
                    split_frag(S[ib], p, hi, lo);
                    const bf16x8 sh = __builtin_bit_cast(bf16x8, hi), sl = __builtin_bit_cast(bf16x8, lo);
                    const bf16x8 k0 = frag_perm(K, LD, n, 32 * ib + 16 * p, half), k1 = frag_perm(K, LD, 32 + n, 32 * ib + 16 * p, half);
                    R[0] = mfma(k0, sh, R[0]);
                    R[1] = mfma(k1, sh, R[1]);
                    R[0] = mfma(k0, sl, R[0]);
                    R[1] = mfma(k1, sl, R[1]);
                    if (MODE == 0) {
                        const bf16x8 q0 = frag_perm(Q, LD, n, 32 * ib + 16 * p, half), q1 = frag_perm(Q, LD, 32 + n, 32 * ib + 16 * p, half);
                        O[0] = mfma(sh, q0, O[0]);
                        O[1] = mfma(sh, q1, O[1]);
                        O[0] = mfma(sl, q0, O[0]);
                        O[1] = mfma(sl, q1, O[1]);
                    }
                }
            if (DEC && MODE == 0) {
                _Pragma("unroll") for (int jb = 0; jb < 2; ++jb) {
                    const float w = __expf(bs[32 * jb + n]);
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) O[jb][x] *= w;
                }
            }
            fresh();
            // R = b V - beta Gamma K S, U = R + (T - I) R: what is not multiplied is not split either
            _Pragma("unroll") for (int kr = 0; kr < 4; ++kr) {
                f32x16& Rb = R[kr >> 1];
                const int x0 = 8 * (kr & 1);
                float w[8], wv[8];
                row_weights(ne, 16 * kr, half, w);
                _Pragma("unroll") for (int x = 0; x < 8; ++x) Rb[x0 + x] *= w[x];
                if (MODE != 2) {
                    row_weights(bb, 16 * kr, half, wv);
                    const u32x4 v8 = __builtin_bit_cast(u32x4, frag_tr_perm(V, LD, 16 * kr, 32 * wave, lane));
                    _Pragma("unroll") for (int e = 0; e < 4; ++e) {
                        Rb[x0 + 2 * e] = fmaf(wv[2 * e], bf16_lo(v8[e]), Rb[x0 + 2 * e]);
                        Rb[x0 + 2 * e + 1] = fmaf(wv[2 * e + 1], bf16_hi(v8[e]), Rb[x0 + 2 * e + 1]);
                    }
                }
            }
            // (U[1] = R[1] here, as U[0], spills 6 registers with a decay: 16 x 16 sequences of 2048, forward, 257 us, this 251; and with
            // U[0] complete before the later rows are split 247)
            f32x16 U[2] = {R[0], f32x16{0}};
            _Pragma("unroll") for (int kr = 0; kr < 4; ++kr) {
                u32x4 hi, lo;
                split_frag(R[kr >> 1], kr & 1, hi, lo);
                const bf16x8 rh = __builtin_bit_cast(bf16x8, hi), rl = __builtin_bit_cast(bf16x8, lo);
                _Pragma("unroll") for (int tb = kr >> 1; tb < 2; ++tb) {
                    const bf16x8 th = frag_tr_perm(Th, LDP, 16 * kr, 32 * tb, lane), tl = frag_tr_perm(Tl, LDP, 16 * kr, 32 * tb, lane);
                    U[tb] = mfma(th, rh, U[tb]);
                    U[tb] = mfma(tl, rh, U[tb]);
                    U[tb] = mfma(th, rl, U[tb]);
                }
                if (kr == 1) asm volatile("" : "+v"(U[0]));
            }
            _Pragma("unroll") for (int x = 0; x < 16; ++x) U[1][x] += R[1][x];
            u32x4 uh[4], ul[4];
            _Pragma("unroll") for (int kr = 0; kr < 4; ++kr) split_frag(U[kr >> 1], kr & 1, uh[kr], ul[kr]);
            __syncthreads();  // (C) scores are in LDS; Q, V and T are spent
            fresh();
            if (MODE == 0) {
                // O^T[v][j] += sum_{r <= j} U^T[v][r] P[j][r]
                _Pragma("unroll") for (int jb = 0; jb < 2; ++jb) {
                    _Pragma("unroll") for (int kr = 0; kr < 2 * (jb + 1); ++kr) {  // keys r >= 32 never reach queries j < 32
                        const bf16x8 ph = frag_perm(Ph, LDP, 32 * jb + n, 16 * kr, half), pl = frag_perm(Pl, LDP, 32 * jb + n, 16 * kr, half);
                        const bf16x8 h = __builtin_bit_cast(bf16x8, uh[kr]), l = __builtin_bit_cast(bf16x8, ul[kr]);
                        O[jb] = mfma(h, ph, O[jb]);
                        O[jb] = mfma(l, ph, O[jb]);
                        O[jb] = mfma(h, pl, O[jb]);
                    }
                    store_packed(stage, LD, 32 * jb + n, 32 * wave, half, pack_block(O[jb]));
                }
                if (a.usave) {
                    _Pragma("unroll") for (int kr = 0; kr < 4; ++kr) {
                        store_frag_rows(Us + 16 * kr * LD + 32 * wave, LD, uh[kr], n, half);
                        store_frag_rows(Usl + 16 * kr * LD + 32 * wave, LD, ul[kr], n, half);
                    }
                }
            }
            fresh();
            // S[i][v] = e^{b_C} S[i][v] + sum_t k_t[i] (wo_t U[t][v])
            if (DEC) {
                const float lam = __expf(bs[C]);
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) S[ib][x] *= lam;
            }
            _Pragma("unroll") for (int kr = 0; kr < 4; ++kr) {
                u32x4 hi = uh[kr], lo = ul[kr];
                if (DEC) {
                    float w[8];
                    row_weights(wo, 16 * kr, half, w);
                    _Pragma("unroll") for (int x = 0; x < 8; ++x) U[kr >> 1][8 * (kr & 1) + x] *= w[x];
                    split_frag(U[kr >> 1], kr & 1, hi, lo);
                }
                const bf16x8 h = __builtin_bit_cast(bf16x8, hi), l = __builtin_bit_cast(bf16x8, lo);
                bf16x8 ka[4];
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) ka[ib] = frag_tr_perm(K, LD, 16 * kr, 32 * ib, lane);
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = mfma(ka[ib], h, S[ib]);
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = mfma(ka[ib], l, S[ib]);
            }
        }
        __syncthreads();  // (E) the last chunk's results are staged
        if (MODE != 0) walk_state_store(S, a.sum + (size_t(seq) * a.nseg + seg) * D * D, false, wave, n, half);
        else if (a.edge_out && seg == nsq - 1) walk_state_store(S, a.edge_out + size_t(seq) * D * D, false, wave, n, half);
    } else {
        TileRegs rq, rk, rv;
        u32x4 rt[3];
        float gval = 0.f, bval = 1.f, bwval = 1.f;
        auto pos = [&](int kk) { return walk_pos(d, walk, kbeg + min(kk, cnt - 1)); };
        auto gload = [&](int kk) {
            const ChunkPos p = pos(kk);
            const size_t pt = p.tok0 + size_t(min(lane, p.L - 1)) * p.ts;
            if (DEC) gval = a.log_alpha[pt];
            if (a.beta) bval = a.beta[pt];
            if (MODE != 2 && a.bw) bwval = a.bw[pt];
            if (MODE == 0) walk_gload<false, kThreads>(rq, a.q, p.tok0, p.ts, p.L, t256);
            walk_gload<false, kThreads>(rk, a.k, p.tok0, p.ts, p.L, t256);
            if (MODE != 2) walk_gload<false, kThreads>(rv, a.v, p.tok0, p.ts, p.L, t256);
            _Pragma("unroll") for (int it = 0; it < 3; ++it)
                rt[it] = *reinterpret_cast<const u32x4*>(a.tt + p.slot * kDeltaT + 8 * (t256 + kThreads * it));
        };
        auto commit = [&](int kk) {
            const int L = pos(kk).L;
            if (MODE == 0) walk_commit<kThreads>(Q, rq, L, t256);
            walk_commit<kThreads>(K2 + (kk & 1) * C * LD, rk, L, t256);
            if (MODE != 2) walk_commit<kThreads>(V, rv, L, t256);
            _Pragma("unroll") for (int it = 0; it < 3; ++it) *reinterpret_cast<u32x4*>(Th + delta_t_place(t256 + kThreads * it)) = rt[it];
            float* bs = tab + (kk & 1) * kDeltaTab;
            float *wo = bs + C + 4, *ne = wo + C, *bb = ne + C;
            if (wave == 0) {
                float gam = 1.f;
                if (DEC) {
                    walk_decay_tables<false, false>(gval, L, 0.f, bs, wo, lane);
                    gam = __expf(bs[lane]);
                }
                ne[lane] = lane < L ? -bval * gam : 0.f;
                bb[lane] = lane < L ? bwval : 0.f;
            }
        };
        auto store = [&](int kk) {  // a chunk's output and pseudo-values
            const ChunkPos p = pos(kk);
            if (a.out) walk_store<false, kThreads>(a.out, stage, p.tok0, p.ts, p.L, t256);
            if (a.usave) {
                walk_store<false, kThreads>(a.usave, Us, p.tok0, p.ts, p.L, t256);
                walk_store<false, kThreads>(a.usave_l, Usl, p.tok0, p.ts, p.L, t256);
            }
        };
        if (cnt > 0) {
            gload(0);
            commit(0);
            if (cnt > 1) gload(1);
        }
        for (int kk = 0; kk < cnt; ++kk) {
            __syncthreads();  // (A)
            if (MODE == 0) {
                walk_scores<DEC>(K2 + (kk & 1) * C * LD, Q, Ph, Pl, tab + (kk & 1) * kDeltaTab, wave, n, half);
                if (kk > 0) store(kk - 1);
            }
            __syncthreads();  // (C)
            if (kk + 1 < cnt) {
                commit(kk + 1);
                if (kk + 2 < cnt) gload(kk + 2);
            }
        }
        __syncthreads();  // (E)
        if (MODE == 0 && cnt > 0) store(cnt - 1);
    }
}

// Entry state of every segment: E_0 = M_0, E_{s+1} = A_s E_s + B_s (REV: from the last segment down, for the state
// gradients, with the transposes of the forward walk's factors), the product on the matrix cores with both factors as bf16 head + remainder (three products; about 2^-16 relative).
// LDS: A head | A remainder (128 x LD each) | E head | E remainder (128 x LDE each).   grid: (4, seqs)
// The value columns of E evolve independently: a workgroup chains 32 of them, A and B of the next segment requested while
// this one is multiplied.  Bound by the latency of that chain: 16 sequences of 2000 tokens in 16
// segments, 0.144 ms with one workgroup per sequence and nothing requested ahead, 0.046 ms so.
constexpr int LDE = 40;  // row stride of a 128 x 32 slice of E
constexpr int kDeltaCombineLds = 2 * D * LD * 2 + 2 * D * LDE * 2;
template <bool REV>
__global__ __launch_bounds__(kThreads, 1) void mk_delta_combine(Dims d, const float* __restrict__ edge_in, const float* __restrict__ sumA,
                                                                const float* __restrict__ sumB, float* __restrict__ bound, int m,
                                                                int nseg) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* Ah = reinterpret_cast<uint16_t*>(smem);
    uint16_t* Al = Ah + D * LD;
    uint16_t* Eh = Al + D * LD;
    uint16_t* El = Eh + D * LDE;
    const int v0 = 32 * blockIdx.x, seq = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, half = lane >> 5;
    const SeqWalk walk = seq_walk(d, seq);
    const int nsq = max(1, (walk.n + m - 1) / m);
    const float* e0 = edge_in ? edge_in + size_t(seq) * D * D : nullptr;
    float* b = bound + size_t(seq) * nseg * D * D;
    // the walk's first segment (REV: the last in time) starts from the edge state; the same as a tile
    float* b0 = b + size_t(REV ? nsq - 1 : 0) * D * D;
    _Pragma("unroll") for (int it = 0; it < 4; ++it) {
        const int p = tid + kThreads * it, row = p >> 3, c4 = p & 7;
        const float4 x = e0 ? *reinterpret_cast<const float4*>(e0 + row * D + v0 + 4 * c4) : float4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<float4*>(b0 + row * D + v0 + 4 * c4) = x;
        const uint32_t h0 = pack2(x.x, x.y), h1 = pack2(x.z, x.w);
        *reinterpret_cast<u32x2*>(Eh + row * LDE + 4 * c4) = u32x2{h0, h1};
        *reinterpret_cast<u32x2*>(El + row * LDE + 4 * c4) =
            u32x2{pack2(x.x - bf16_lo(h0), x.y - bf16_hi(h0)), pack2(x.z - bf16_lo(h1), x.w - bf16_hi(h1))};
    }
    if (nsq <= 1) return;
    float4 ra[16];  // A of the next segment: 128 x 128 floats by 256 threads, 4 at a time
    f32x16 rb;      // its B, at the result registers: rows 32 w .. + 31, this workgroup's columns
    auto gload = [&](int st) {
        const int s = REV ? nsq - 1 - min(st, nsq - 2) : min(st, nsq - 2);
        const size_t slot = (size_t(seq) * nseg + s) * D * D;
        _Pragma("unroll") for (int it = 0; it < 16; ++it) {
            const int p = tid + kThreads * it;
            ra[it] = *reinterpret_cast<const float4*>(sumA + slot + (p >> 5) * D + 4 * (p & 31));
        }
        _Pragma("unroll") for (int x = 0; x < 16; ++x)
            rb[x] = sumB[slot + size_t(32 * wave + 8 * (x >> 2) + 4 * half + (x & 3)) * D + v0 + n];
    };
    gload(0);
    for (int st = 0; st + 1 < nsq; ++st) {
        const int s = REV ? nsq - 1 - st : st;   // the segment walked in this step; its end state enters segment s -+ 1
        _Pragma("unroll") for (int it = 0; it < 16; ++it) {
            const int p = tid + kThreads * it, row = p >> 5, c4 = p & 31;
            const float4 x = ra[it];
            const uint32_t h0 = pack2(x.x, x.y), h1 = pack2(x.z, x.w);
            *reinterpret_cast<u32x2*>(Ah + row * LD + 4 * c4) = u32x2{h0, h1};
            *reinterpret_cast<u32x2*>(Al + row * LD + 4 * c4) =
                u32x2{pack2(x.x - bf16_lo(h0), x.y - bf16_hi(h0)), pack2(x.z - bf16_lo(h1), x.w - bf16_hi(h1))};
        }
        f32x16 acc = rb;
        gload(st + 1);
        __syncthreads();  // A and E tiles are complete
        // E'[i][v] = sum_j A[i][j] E[j][v] + B[i][v]
        _Pragma("unroll") for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 ah = REV ? frag_tr(Ah, LD, 16 * ks, 32 * wave, lane) : frag(Ah, LD, 32 * wave + n, 16 * ks + 8 * half);
            const bf16x8 al = REV ? frag_tr(Al, LD, 16 * ks, 32 * wave, lane) : frag(Al, LD, 32 * wave + n, 16 * ks + 8 * half);
            const bf16x8 eh = frag_tr(Eh, LDE, 16 * ks, 0, lane), el = frag_tr(El, LDE, 16 * ks, 0, lane);
            acc = mfma(ah, eh, acc);
            acc = mfma(ah, el, acc);
            acc = mfma(al, eh, acc);
        }
        __syncthreads();  // every wave has read A and E
        float* out = b + size_t(REV ? s - 1 : s + 1) * D * D;
        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
            const int i = 32 * wave + 8 * (x >> 2) + 4 * half + (x & 3);
            const float e = acc[x];
            out[size_t(i) * D + v0 + n] = e;
            const uint32_t h = pack2(e, 0.f);
            Eh[i * LDE + n] = uint16_t(h & 0xffffu);
            El[i * LDE + n] = uint16_t(pack2(e - bf16_lo(h), 0.f) & 0xffffu);
        }
        // the barrier at the top of the next step orders the writes of A and E
    }
}

// ---------------------------------------------------------------------------------------------
// Backward.  With U known, M_t = alpha_t M_{t-1} + k_t^T u_t is the scalar-decay recurrence on values U, so most of the
// adjoint is the diagonal kinds' - if the state gradients are the delta rule's.  Those carry a feedback term, because u_t
// depends on the state the chunk starts from: R = (I + L) U = diag(b) V - diag(beta Gamma) K S.  Per chunk, with A the masked
// decayed scores, dS' the gradient of the state at the chunk end and W the gradient of R,
//     dU = A^T dO + diag(wo) K dS' ,   W = T^T dU ,
//     dS = Gamma_C dS' + (diag(Gamma) Q)^T dO - (diag(beta Gamma) K)^T W .
// Everything that reaches the inputs through the solve follows from W without T (the gradient of T is dU R^T and
// dL = -T^T (dU R^T) T^T = -W U^T, since T R = U):
//     dv_t = b_t W_t ,  db_t = W_t . v_t ,
//     X_t = -Gamma_t S W_t + sum_{r < t} H_tr k_r ,   H_tr = -D_tr (W_t . u_r) ,  D_tr = e^{lg_t - lg_r} ,
//     dk_t += beta_t X_t + sum_{j > t} beta_j H_jt k_j ,   d beta_t = k_t . X_t ,
// and the erase term enters the decay gradient like a second query: + beta_t k_t . X_t, its key side with the other
// key gradients.  mk_delta_rwalk walks a sequence backward with dS in the accumulators (the forward walker's block layout),
// stores dS' per chunk in the fragment-major bf16 form the gradient walker reads, W as bf16 head + remainder, dv and db; the
// gradient walker (VSPLIT) does the rest, entering its segments with the forward walk's states.  Bytes a token of the backward:
// 5.1 KB.  With dU handed on instead of W, a kernel of its own took the gradient through T chunk by chunk (9.2 KB a token, a
// summary pass over U for the entry states): forward + backward, 16 x 16 sequences of 2048, 1.64 -> 1.19 ms.
struct DeltaRevArgs {
    const uint16_t *q, *k, *v, *d_o;
    const uint16_t* tt;       // [BH*N][kDeltaT]
    const float *log_alpha, *beta, *bw;
    uint16_t* dstates;        // [BH*N] fragment-major bf16: slot c = gradient of the state at the end of chunk c
    uint16_t *w_h, *w_l;      // [BH*T][128] bf16 (library order)
    uint16_t* dv;             // layout of v
    float* d_bw;              // per token, may be NULL
    const float* edge_in;     // d M_T [i][v] per sequence or NULL
    float* edge_out;          // d M_0 or NULL
    int m, nseg;              // segments as for the forward walker: the walk enters segment s (from above) with bound[seq][s],
    const float* bound;       // the summary leaves what the segment makes of a zero state in sum[seq][s] (what it makes of the
    float* sum;               // identity is the transpose of the forward walk's factor)
};
// LDS: Q | K | dO (64 x LD) | T^T head | remainder | scores head | remainder (64 x LDP) | stage of dS' (bf16, 128 x LD) | stage of
// W (fp32, 64 x LDW) | two sets of (bs, wo, Gamma, -beta Gamma, b)
constexpr int LDW = D + 4;
constexpr int kDeltaRevTab = 5 * C + 4;
constexpr int kDeltaRevLds = (3 * C * LD + 4 * C * LDP + D * LD) * 2 + (C * LDW + 2 * kDeltaRevTab) * 4;
static_assert(kDeltaRevLds <= 160 * 1024, "one workgroup's LDS");

// grid: (segments, seqs).  SUM: summary of a segment from a zero state (nothing stored but its end state).  Eight waves, two per
// SIMD, split by function as in the forward walk:
//   waves 0..3 carry the state (wave w: value columns [32 w, 32 w + 32) of dS, dU and W): the chain dU, W, state update.  The
//              products that lead from one to the next take the block before straight out of the accumulators (lane = value
//              column, registers = the next contraction's index), so only scores, T and input rows are read from LDS;
//   waves 4..7 the scores, the tables, and what leaves: dS' (staged while dU's state part is formed) and, a chunk later, W, dv and db.
// All share the rows on their way in.  16 x 16 sequences of 2048, 2.5 KB a token: 380 us with four waves
// doing everything in turn, 321 so.
template <bool DEC, bool SUM>
__global__ __launch_bounds__(512, 1) void mk_delta_rwalk(Dims d, DeltaRevArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* Q = reinterpret_cast<uint16_t*>(smem);
    uint16_t* K = Q + C * LD;
    uint16_t* dO = K + C * LD;
    uint16_t* TTh = dO + C * LD;
    uint16_t* TTl = TTh + C * LDP;
    uint16_t* Ph = TTl + C * LDP;
    uint16_t* Pl = Ph + C * LDP;
    uint16_t* dSt = Pl + C * LDP;
    float* Ws = reinterpret_cast<float*>(dSt + D * LD);
    float* tab = Ws + C * LDW;

    const int seg = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3;
    int lane = tid & 63, n = lane & 31, half = lane >> 5;
    auto fresh = [&]() {  // (as in mk_walk_grad)
        asm volatile("" : "+v"(lane));
        n = lane & 31;
        half = lane >> 5;
    };
    const int t256 = tid & 255;
    const bool carrier = wave8 < 4;
    const SeqWalk walk = seq_walk(d, seq);
    const int nsq = max(1, (walk.n + a.m - 1) / a.m);
    const int kbeg = seg * a.m, kend = min(walk.n, kbeg + a.m), cnt = max(kend - kbeg, 0);
    if (SUM) {
        if (cnt <= 0 || seg == 0) return;  // only segments whose end state (backward in time) another one starts from
    } else if (seg >= nsq) {
        return;
    }
    auto pos = [&](int kk) { return walk_pos(d, walk, kend - 1 - min(kk, cnt - 1)); };
    TileRegs rq, rk, ro;
    auto gload_rows = [&](const ChunkPos& p) {
        walk_gload<false, 512>(rq, a.q, p.tok0, p.ts, p.L, tid);
        walk_gload<false, 512>(ro, a.d_o, p.tok0, p.ts, p.L, tid);
        walk_gload<false, 512>(rk, a.k, p.tok0, p.ts, p.L, tid);
    };
    auto commit_rows = [&](int L) {
        walk_commit<512>(Q, rq, L, tid);
        walk_commit<512>(dO, ro, L, tid);
        walk_commit<512>(K, rk, L, tid);
    };

    if (carrier) {
        f32x16 S[4];  // dS[ib][4g+j] = dS[i = 32 ib + 8g + 4 half + j][v = 32 wave + n]
        _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = f32x16{0};
        if (!SUM) {
            const float* ein = a.nseg > 1 ? a.bound + (size_t(seq) * a.nseg + seg) * D * D
                                          : (a.edge_in ? a.edge_in + size_t(seq) * D * D : nullptr);
            if (ein) walk_state_load(S, ein, false, wave, n, half);
        }
        if (cnt > 0) gload_rows(pos(0));
        for (int kk = 0; kk < cnt; ++kk) {
            const float* bs = tab + (kk & 1) * kDeltaRevTab;
            const float *wo = bs + C + 4, *gm = wo + C, *ne = gm + C;
            commit_rows(pos(kk).L);
            if (kk + 1 < cnt) gload_rows(pos(kk + 1));
            __syncthreads();  // (A) tiles and tables of this chunk are in LDS
            fresh();
            // dU[t][v] = wo_t sum_i k_t[i] dS'[i][v] + sum_{j >= t} P[j][t] dO[j][v]; dS' leaves as its bf16 heads
            f32x16 dU[2] = {{0}, {0}};
            _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
                _Pragma("unroll") for (int p = 0; p < 2; ++p) {
                    u32x4 hi, lo;
                    split_frag(S[ib], p, hi, lo);
                    const bf16x8 sh = __builtin_bit_cast(bf16x8, hi), sl = __builtin_bit_cast(bf16x8, lo);
                    const bf16x8 k0 = frag_perm(K, LD, n, 32 * ib + 16 * p, half), k1 = frag_perm(K, LD, 32 + n, 32 * ib + 16 * p, half);
                    dU[0] = mfma(k0, sh, dU[0]);
                    dU[1] = mfma(k1, sh, dU[1]);
                    dU[0] = mfma(k0, sl, dU[0]);
                    dU[1] = mfma(k1, sl, dU[1]);
                    if (!SUM) store_frag_rows(dSt + (32 * ib + 16 * p) * LD + 32 * wave, LD, hi, n, half);
                }
            if (DEC) {
                _Pragma("unroll") for (int kt = 0; kt < 4; ++kt) {
                    float w[8];
                    row_weights(wo, 16 * kt, half, w);
                    _Pragma("unroll") for (int x = 0; x < 8; ++x) dU[kt >> 1][8 * (kt & 1) + x] *= w[x];
                }
            }
            __syncthreads();  // (C) the scores and the stage of dS' are in LDS
            fresh();
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 dot = frag_tr(dO, LD, 16 * ks, 32 * wave, lane);
                _Pragma("unroll") for (int tb = 0; tb <= (ks >> 1); ++tb) {  // queries j < 32 never see keys t >= 32
                    dU[tb] = mfma(frag_tr(Ph, LDP, 16 * ks, 32 * tb, lane), dot, dU[tb]);
                    dU[tb] = mfma(frag_tr(Pl, LDP, 16 * ks, 32 * tb, lane), dot, dU[tb]);
                }
            }
            // W[r][v] = dU[r][v] + sum_{t > r} T[t][r] dU[t][v]
            f32x16 W[2] = {dU[0], dU[1]};
            _Pragma("unroll") for (int kt = 0; kt < 4; ++kt) {
                u32x4 hi, lo;
                split_frag(dU[kt >> 1], kt & 1, hi, lo);
                const bf16x8 uh = __builtin_bit_cast(bf16x8, hi), ul = __builtin_bit_cast(bf16x8, lo);
                _Pragma("unroll") for (int rb = 0; rb <= (kt >> 1); ++rb) {
                    const bf16x8 th = frag_perm(TTh, LDP, 32 * rb + n, 16 * kt, half), tl = frag_perm(TTl, LDP, 32 * rb + n, 16 * kt, half);
                    W[rb] = mfma(th, uh, W[rb]);
                    W[rb] = mfma(tl, uh, W[rb]);
                    W[rb] = mfma(th, ul, W[rb]);
                }
            }
            fresh();
            if (!SUM) {
                _Pragma("unroll") for (int rb = 0; rb < 2; ++rb)
                    _Pragma("unroll") for (int x = 0; x < 16; ++x)
                        Ws[(32 * rb + 8 * (x >> 2) + 4 * half + (x & 3)) * LDW + 32 * wave + n] = W[rb][x];
            }
            // dS = Gamma_C dS' + sum_t (Gamma_t q_t)^T dO_t - sum_t (beta_t Gamma_t k_t)^T W_t
            if (DEC) {
                const float lam = __expf(bs[C]);
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) S[ib][x] *= lam;
            }
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
                const u32x4 raw = __builtin_bit_cast(u32x4, frag_tr(dO, LD, 16 * ks, 32 * wave, lane));
                u32x4 hi = raw, lo = {0, 0, 0, 0};
                if (DEC) {
                    const float4 w0 = *reinterpret_cast<const float4*>(gm + 16 * ks + 8 * half);
                    const float4 w1 = *reinterpret_cast<const float4*>(gm + 16 * ks + 8 * half + 4);
                    const float w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                    _Pragma("unroll") for (int p = 0; p < 4; ++p) {
                        const float x0 = bf16_lo(raw[p]) * w[2 * p], x1 = bf16_hi(raw[p]) * w[2 * p + 1];
                        hi[p] = pack2(x0, x1);
                        lo[p] = pack2(x0 - bf16_lo(hi[p]), x1 - bf16_hi(hi[p]));
                    }
                }
                const bf16x8 oh = __builtin_bit_cast(bf16x8, hi), ol = __builtin_bit_cast(bf16x8, lo);
                float w[8];
                row_weights(ne, 16 * ks, half, w);
                f32x16& Wb = W[ks >> 1];
                _Pragma("unroll") for (int x = 0; x < 8; ++x) Wb[8 * (ks & 1) + x] *= w[x];
                split_frag(Wb, ks & 1, hi, lo);
                const bf16x8 eh = __builtin_bit_cast(bf16x8, hi), el = __builtin_bit_cast(bf16x8, lo);
                _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) {
                    const bf16x8 qa = frag_tr(Q, LD, 16 * ks, 32 * ib, lane);
                    S[ib] = mfma(qa, oh, S[ib]);
                    if (DEC) S[ib] = mfma(qa, ol, S[ib]);
                    const bf16x8 ka = frag_tr_perm(K, LD, 16 * ks, 32 * ib, lane);
                    S[ib] = mfma(ka, eh, S[ib]);
                    S[ib] = mfma(ka, el, S[ib]);
                }
            }
            __syncthreads();  // (D) every read of this chunk's tiles is done
            fresh();
        }
        if (SUM) walk_state_store(S, a.sum + (size_t(seq) * a.nseg + seg) * D * D, false, wave, n, half);
        else if (a.edge_out && seg == 0) walk_state_store(S, a.edge_out + size_t(seq) * D * D, false, wave, n, half);
    } else {
        u32x4 rt[3];
        TileRegs rv;
        float gval = 0.f, bval = 1.f, bwval = 1.f;
        auto gload = [&](int kk) {
            const ChunkPos p = pos(kk);
            const size_t pt = p.tok0 + size_t(min(lane, p.L - 1)) * p.ts;
            if (DEC) gval = a.log_alpha[pt];
            if (a.beta) bval = a.beta[pt];
            if (!SUM && a.bw) bwval = a.bw[pt];
            gload_rows(p);
            _Pragma("unroll") for (int it = 0; it < 3; ++it) rt[it] = *reinterpret_cast<const u32x4*>(a.tt + p.slot * kDeltaT + 8 * (t256 + kThreads * it));
        };
        // W of the kk-th chunk to memory, and dv and db on the way (rv: the chunk's rows of v, in the same pieces)
        auto leave = [&](int kk) {
            const ChunkPos p = pos(kk);
            const float* bb = tab + (kk & 1) * kDeltaRevTab + 4 * C + 4;
            _Pragma("unroll") for (int it = 0; it < 4; ++it) {
                const int q = t256 + kThreads * it, row = q >> 4, piece = q & 15;
                const float4 x0 = *reinterpret_cast<const float4*>(Ws + row * LDW + 8 * piece), x1 = *reinterpret_cast<const float4*>(Ws + row * LDW + 8 * piece + 4);
                const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w}, b = bb[row];
                u32x4 h, l, o;
                float s = 0.f;
                _Pragma("unroll") for (int e = 0; e < 4; ++e) {
                    h[e] = pack2(x[2 * e], x[2 * e + 1]);
                    l[e] = pack2(x[2 * e] - bf16_lo(h[e]), x[2 * e + 1] - bf16_hi(h[e]));
                    o[e] = pack2(b * x[2 * e], b * x[2 * e + 1]);
                    s += x[2 * e] * bf16_lo(rv.v[it][e]) + x[2 * e + 1] * bf16_hi(rv.v[it][e]);
                }
                if (row < p.L) {
                    const size_t off = (p.wtok0 + row) * D + 8 * piece, tok = p.tok0 + size_t(row) * p.ts;
                    *reinterpret_cast<u32x4*>(a.w_h + off) = h;
                    *reinterpret_cast<u32x4*>(a.w_l + off) = l;
                    __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(a.dv + tok * D + 8 * piece));
                }
                _Pragma("unroll") for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
                if (a.d_bw && piece == 0 && row < p.L) a.d_bw[p.tok0 + size_t(row) * p.ts] = s;
            }
        };
        if (cnt > 0) gload(0);
        for (int kk = 0; kk < cnt; ++kk) {
            const ChunkPos cp = pos(kk);
            float* bs = tab + (kk & 1) * kDeltaRevTab;
            float *wo = bs + C + 4, *gm = wo + C, *ne = gm + C, *bb = ne + C;
            commit_rows(cp.L);
            _Pragma("unroll") for (int it = 0; it < 3; ++it) *reinterpret_cast<u32x4*>(TTh + delta_t_place(t256 + kThreads * it)) = rt[it];
            if (wave == 0) {
                float gam = 1.f;
                if (DEC) {
                    walk_decay_tables<false, false>(gval, cp.L, 0.f, bs, wo, lane);
                    gm[lane] = gam = __expf(bs[lane]);
                }
                ne[lane] = lane < cp.L ? -bval * gam : 0.f;
                bb[lane] = lane < cp.L ? bwval : 0.f;
            }
            if (kk + 1 < cnt) gload(kk + 1);
            __syncthreads();  // (A)
            walk_scores<DEC>(K, Q, Ph, Pl, bs, wave, n, half);
            if (!SUM && kk > 0) leave(kk - 1);
            __syncthreads();  // (C)
            if (!SUM) {
                walk_gload<false, kThreads>(rv, a.v, cp.tok0, cp.ts, cp.L, t256);
                uint16_t* dst = a.dstates + cp.slot * D * D;
                _Pragma("unroll") for (int ks = 0; ks < 8; ++ks)
                    __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(dSt + (32 * wave + n) * LD + 16 * ks + 8 * half),
                                                reinterpret_cast<u32x4*>(dst + state_frag_off(wave, ks, lane)));
            }
            __syncthreads();  // (D)
        }
        if (!SUM && cnt > 0) leave(cnt - 1);
    }
}
