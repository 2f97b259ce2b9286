// Fused chunk walkers of the scalar decay kinds (none / per head / per token): bf16 operands, fp32
// accumulation, chunk = 64, d_k = d_v = 128.  Included by lsm_mfma.hip.
//
// One workgroup walks a run of consecutive chunks (a "segment") of one (b,h) recurrence with the
// 128 x 128 state in MFMA accumulators, so the forward pass writes no per-chunk state at all and the
// backward pass only the state gradients.  Per chunk the forward walker evaluates Algorithm 2 of the
// paper with the decay folded in,
//     o_t = e^{b_t} q_t S + sum_{r <= t} (q_t . k_r) e^{b_t - b_r} v_r        (O_inter + O_intra)
//     S  <- e^{b_C} S + sum_r e^{b_C - b_r} k_r^T v_r                         (chunk state, prefix)
// and the gradient walker (further down) the adjoint of the same chunk with S carried the same way.
//
// Segments: with fewer recurrences than the chip can keep busy a sequence is cut into segments of m
// chunks.  A first pass (SUMMARY: the state update alone, from a zero state) leaves each segment's own
// contribution and total log-decay, a small scan turns them into the state every segment starts from,
// and the walkers then run all segments in parallel.  Only those entry states (one per m chunks) ever
// reach memory.  REV walks backward in time (a chunk's rows are loaded in reverse token order and beta
// is the exclusive instead of the inclusive running sum of the log-decays in walk order); it serves
// the summary pass of the reverse direction.
#pragma once

struct WalkArgs {
    const uint16_t *xq, *xk, *xv;  // rows in the query, key and value role (forward pass: q, k, v)
    const float* g;                // log-decay (per kind)
    uint16_t* out;
    const float* edge_in;  // state a whole sequence starts from, [i][v] fp32 per sequence; NULL = zero
    float* edge_out;       // state it ends with; NULL = not wanted
    float* bound;          // [slot][128 x 128] fp32, [i][v]: entry state of every segment but the first (nseg > 1; bound_slot())
    float* gseg;           // [slot]: total log-decay of each segment (SUMMARY writes)
    int m, nseg;           // chunks per segment, segments per sequence (upper bound for packed input)
    int skip;              // SUMMARY, REV: segments [0, skip) feed no other walk and are left out (at least 1)
};

// tile rows in walk order: row r holds token r (forward) or token L-1-r (backward); rows >= L are zero.
// NT threads share a tile: 1024 / NT pieces of 16 bytes each.
template <bool REV, int NT>
__device__ __forceinline__ void walk_gload(TileRegs& r, const uint16_t* src, size_t tok0, int ts, int L, int tid) {
    // uniform base (scalar registers) + a 32-bit byte offset per lane, shared by every tile of the chunk
    const char* base = reinterpret_cast<const char*>(src + tok0 * D);
    _Pragma("unroll") for (int it = 0; it < 1024 / NT; ++it) {
        const int p = tid + NT * it, row = min(p >> 4, L - 1), cp = p & 15;
        const int tok = REV ? L - 1 - row : row;
        const uint32_t off = (uint32_t(tok) * uint32_t(ts) * D + cp * 8) * 2;
        r.v[it] = *reinterpret_cast<const u32x4*>(base + off);
    }
}
template <int NT>
__device__ __forceinline__ void walk_commit(uint16_t* dst, const TileRegs& r, int L, int tid) {
    _Pragma("unroll") for (int it = 0; it < 1024 / NT; ++it) {
        const int p = tid + NT * it, row = p >> 4, cp = p & 15;
        const uint32_t keep = row < L ? 0xffffffffu : 0u;
        *reinterpret_cast<u32x4*>(dst + row * LD + cp * 8) = u32x4{r.v[it].x & keep, r.v[it].y & keep, r.v[it].z & keep, r.v[it].w & keep};
    }
}
// NT threads store an output stage
template <bool REV, int NT = kThreads>
__device__ __forceinline__ void walk_store(uint16_t* dst, const uint16_t* src, size_t tok0, int ts, int L, int tid) {
    char* base = reinterpret_cast<char*>(dst + tok0 * D);
    _Pragma("unroll") for (int it = 0; it < 1024 / NT; ++it) {
        const int p = tid + NT * it, row = p >> 4, cp = p & 15;
        const uint32_t off = (uint32_t(REV ? L - 1 - row : row) * uint32_t(ts) * D + cp * 8) * 2;
        if (row < L)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(src + row * LD + cp * 8), reinterpret_cast<u32x4*>(base + off));
    }
}

// B operand whose k order follows a D-layout block used as A operand: slot e of lane (n, half) is
// column col0 + 8 (e / 4) + 4 half + e % 4 of row `row`
__device__ __forceinline__ bf16x8 frag_perm(const uint16_t* tile, int ld, int row, int col0, int half) {
    const u32x2 a = *reinterpret_cast<const u32x2*>(tile + row * ld + col0 + 4 * half);
    const u32x2 b = *reinterpret_cast<const u32x2*>(tile + row * ld + col0 + 8 + 4 * half);
    return __builtin_bit_cast(bf16x8, u32x4{a.x, a.y, b.x, b.y});
}

// mask (key r <= query j) and decay e^{beta_j - beta_r} of a score block whose rows index keys
template <bool DEC>
__device__ __forceinline__ void walk_mask(f32x16& acc, int m0, int ncol, const float* bs, int half) {
    const float bn = DEC ? bs[ncol] : 0.f;
    _Pragma("unroll") for (int g = 0; g < 4; ++g) {
        float bmv[4] = {0.f, 0.f, 0.f, 0.f};
        if (DEC) {
            const float4 bm = *reinterpret_cast<const float4*>(bs + m0 + 8 * g + 4 * half);
            bmv[0] = bm.x; bmv[1] = bm.y; bmv[2] = bm.z; bmv[3] = bm.w;
        }
        _Pragma("unroll") for (int jj = 0; jj < 4; ++jj) {
            const int r = m0 + 8 * g + 4 * half + jj, x = 4 * g + jj;
            const float w = DEC ? __expf(bn - bmv[jj]) : 1.f;
            acc[x] = r <= ncol ? acc[x] * w : 0.f;
        }
    }
}

__host__ __device__ constexpr int walk_lds(bool summary) {
    return summary ? 2 * C * LD * 2 + (2 * C + 8) * 4 : (3 * C * LD + 2 * C * LDP) * 2 + (2 * C + 8) * 4;
}

// D[m][n] = sum_f Am[m0 + m][f] * Bm[n0 + n][f] over the 128 features of two row-major LDS tiles, the
// fragments requested four k-steps at a time (a lower register peak than all sixteen at once)
__device__ __forceinline__ f32x16 score_block2(const uint16_t* Am, int m0, const uint16_t* Bm, int n0, int n, int half) {
    f32x16 acc = {0};
    _Pragma("unroll") for (int h4 = 0; h4 < 2; ++h4) {
        bf16x8 fa[4], fb[4];
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
            fa[ks] = frag(Am, LD, m0 + n, 16 * (4 * h4 + ks) + 8 * half);
            fb[ks] = frag(Bm, LD, n0 + n, 16 * (4 * h4 + ks) + 8 * half);
        }
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) acc = mfma(fa[ks], fb[ks], acc);
    }
    return acc;
}

// ---- the four contractions of one chunk for the wave that owns value features [32 w4, 32 w4 + 32)
// state block ib: S[ib][4g+j] = state[key feature 32 ib + 8g + 4 half + j][value feature 32 w4 + n]

// inter: O^T[v][j] = e^{beta_j} sum_i S[i][v] q_j[i], the state blocks as A operands straight from the
// accumulators (bf16 head + remainder), the query rows read in the matching k order
template <bool DEC>
__device__ __forceinline__ void walk_inter(f32x16 (&O)[2], const f32x16 (&S)[4], const uint16_t* Q, const float* bs, int n, int half) {
    O[0] = f32x16{0};
    O[1] = f32x16{0};
    _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
        _Pragma("unroll") for (int p = 0; p < 2; ++p) {
            u32x4 hi, lo;
            split_frag(S[ib], p, hi, lo);
            const bf16x8 sh = __builtin_bit_cast(bf16x8, hi), sl = __builtin_bit_cast(bf16x8, lo);
            const bf16x8 qf0 = frag_perm(Q, LD, n, 32 * ib + 16 * p, half);
            const bf16x8 qf1 = frag_perm(Q, LD, 32 + n, 32 * ib + 16 * p, half);
            O[0] = mfma(sh, qf0, O[0]);
            O[1] = mfma(sh, qf1, O[1]);
            O[0] = mfma(sl, qf0, O[0]);
            O[1] = mfma(sl, qf1, O[1]);
        }
    if (DEC) {
        _Pragma("unroll") for (int jb = 0; jb < 2; ++jb) {
            const float w = __expf(bs[32 * jb + n]);
            _Pragma("unroll") for (int x = 0; x < 16; ++x) O[jb][x] *= w;
        }
    }
}
// scores: each of the three 32 x 32 blocks on or below the diagonal by one wave (w4 = 0: (0,0), 1: (1,0),
// 2: (1,1)), mask and decay on its accumulators, handed to the others through LDS as head + remainder
template <bool DEC>
__device__ __forceinline__ void walk_scores(const uint16_t* K, const uint16_t* Q, uint16_t* Ph, uint16_t* Pl, const float* bs,
                                            int w4, int n, int half) {
    if (w4 >= 3) return;
    const int pjb = w4 ? 1 : 0, prb = w4 == 2 ? 1 : 0;
    f32x16 P = score_block2(K, 32 * prb, Q, 32 * pjb, n, half);  // D[m = r][n = j] = k_r . q_j
    walk_mask<DEC>(P, 32 * prb, 32 * pjb + n, bs, half);
    store_block_t_split(Ph, Pl, LDP, 32 * pjb + n, 32 * prb, half, P);
}
// intra: O^T[v][j] += sum_{r <= j} V^T[v][r] P[j][r] for the query block jb
__device__ __forceinline__ void walk_intra(f32x16& O, int jb, const uint16_t* V, const uint16_t* Ph, const uint16_t* Pl, int w4,
                                           int lane, int n, int half) {
    const int j = 32 * jb + n;
    _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
        if (ks >= 2 * (jb + 1)) break;  // keys r >= 32 never reach queries j < 32
        const bf16x8 vt = frag_tr(V, LD, 16 * ks, 32 * w4, lane);
        O = mfma(vt, frag(Ph, LDP, j, 16 * ks + 8 * half), O);
        O = mfma(vt, frag(Pl, LDP, j, 16 * ks + 8 * half), O);
    }
}
// state: S[i][v] = e^{b_C} S[i][v] + sum_t K^T[i][t] (wo_t V[t][v]); the weighted value slice of this wave is
// split into head + remainder in registers (wo in tr4_at order).  SCALE = false: the weights already carry every decay.
// K2 (KSPLIT): remainder plane of the key-role tile (remainder x remainder is left out).
template <bool DEC, bool SCALE, bool KSPLIT = false>
__device__ __forceinline__ void walk_update(f32x16 (&S)[4], const uint16_t* K, const uint16_t* V, const float* wo, float bC, int w4,
                                            int lane, int half, const uint16_t* K2 = nullptr) {
    if (DEC && SCALE) {
        const float lam = __expf(bC);
        _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
            _Pragma("unroll") for (int x = 0; x < 16; ++x) S[ib][x] *= lam;
    }
    _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
        const u32x4 raw = __builtin_bit_cast(u32x4, frag_tr4(V, LD, 16 * ks, 32 * w4, lane));
        u32x4 hi = raw, lo = {0, 0, 0, 0};
        if (DEC) {
            const float4 w0 = *reinterpret_cast<const float4*>(wo + 16 * ks + 8 * half);
            const float4 w1 = *reinterpret_cast<const float4*>(wo + 16 * ks + 8 * half + 4);
            const float w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
            _Pragma("unroll") for (int p = 0; p < 4; ++p) {
                const float x0 = bf16_lo(raw[p]) * w[2 * p], x1 = bf16_hi(raw[p]) * w[2 * p + 1];
                hi[p] = pack2(x0, x1);
                lo[p] = pack2(x0 - bf16_lo(hi[p]), x1 - bf16_hi(hi[p]));
            }
        }
        const bf16x8 vh = __builtin_bit_cast(bf16x8, hi), vl = __builtin_bit_cast(bf16x8, lo);
        bf16x8 ka[4];
        _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) ka[ib] = frag_tr4(K, LD, 16 * ks, 32 * ib, lane);
        _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = mfma(ka[ib], vh, S[ib]);
        if (DEC) {
            _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = mfma(ka[ib], vl, S[ib]);
        }
        if (KSPLIT) {
            _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = mfma(frag_tr4(K2, LD, 16 * ks, 32 * ib, lane), vh, S[ib]);
        }
    }
}
// chunk-local decay tables by one wave: beta (inclusive running sum of the log-decays in walk order, exclusive
// when walking backward), b_C, and the weights wo = e^{b_C - beta + extra} of the state update
// (TR4: wo in tr4_at order)
template <bool REV, bool TR4 = true>
__device__ __forceinline__ float walk_decay_tables(float gval, int L, float extra, float* bs, float* wo, int lane) {
    const float x = lane < L ? gval : 0.f;
    float inc = x;
    for (int off = 1; off < 64; off <<= 1) {
        const float y = __shfl_up(inc, off, 64);
        if (lane >= off) inc += y;
    }
    const float bC = __shfl(inc, 63, 64), beta = REV ? inc - x : inc;
    bs[lane] = beta;
    wo[TR4 ? tr4_at(lane) : lane] = __expf(bC - beta + extra);
    if (lane == 0) bs[C] = bC;
    return bC;
}
// state block layout <-> the [i][v] fp32 arrays (transposed: the walker's state is the transpose of the array)
// (erow: row stride of the array; the caller's states have d_v columns, the library's own 128)
__device__ __forceinline__ void walk_state_load(f32x16 (&S)[4], const float* e, bool transposed, int w4, int n, int half, int erow = D) {
    _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
            const int mm = 32 * ib + 8 * (x >> 2) + 4 * half + (x & 3), nn = 32 * w4 + n;
            S[ib][x] = transposed ? e[nn * erow + mm] : e[mm * erow + nn];
        }
}
__device__ __forceinline__ void walk_state_store(const f32x16 (&S)[4], float* e, bool transposed, int w4, int n, int half, int erow = D) {
    _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
        _Pragma("unroll") for (int x = 0; x < 16; ++x) {
            const int mm = 32 * ib + 8 * (x >> 2) + 4 * half + (x & 3), nn = 32 * w4 + n;
            e[transposed ? nn * erow + mm : mm * erow + nn] = S[ib][x];
        }
}
// the caller's state of recurrence `seq` ([d_k][d_v] fp32), at the value slice of this pass
__device__ __forceinline__ size_t edge_off(const Dims& d, int seq) { return (size_t(seq) * D * d.vm + d.vs) * D; }
// REV: walk backward in time.  DEC: a decay is present.  SUMMARY: the state update alone, from a zero
// state, result to a.bound / a.gseg.
template <bool REV, bool DEC, bool SUMMARY>
__device__ __forceinline__ void walk_body(const Dims& d, const WalkArgs& a, const SeqWalk& walk, int seg, unsigned char* smem) {
    // LDS: SUMMARY: K | V | bs | wo;   else: Q | K | V | P head | P remainder | bs | wo
    uint16_t* Q = reinterpret_cast<uint16_t*>(smem);
    uint16_t* K = SUMMARY ? Q : Q + C * LD;
    uint16_t* V = K + C * LD;
    uint16_t* Ph = V + C * LD;
    uint16_t* Pl = Ph + C * LDP;
    float* bs = reinterpret_cast<float*>(SUMMARY ? V + C * LD : Pl + C * LDP);  // beta[64], then b_C
    float* wo = bs + C + 4;                                                      // e^{b_C - beta}[64]
    uint16_t* stage = Q;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 31, half = lane >> 5;
    const int nsq = (walk.n + a.m - 1) / a.m;  // segments of this sequence
    const int kbeg = seg * a.m, kend = min(walk.n, kbeg + a.m), cnt = kend - kbeg;
    const bool empty_seq = walk.n == 0 && seg == 0;  // packed input: the state passes through
    if (SUMMARY) {
        // only segments whose end state another segment starts from
        if (cnt <= 0 || (REV ? seg < a.skip : seg >= nsq - 1)) return;
    } else if (cnt <= 0 && !empty_seq) {
        return;
    }
    const bool last = empty_seq || (REV ? seg == 0 : seg == nsq - 1);  // this walk ends the sequence

    f32x16 S[4];
    _Pragma("unroll") for (int ib = 0; ib < 4; ++ib) S[ib] = f32x16{0};
    if (!SUMMARY) {
        if (seg > 0) walk_state_load(S, a.bound + (bound_slot(d, walk, a.m, a.nseg) + seg) * D * D, false, wave, n, half);
        else if (a.edge_in) walk_state_load(S, a.edge_in + edge_off(d, walk.edge), false, wave, n, half, D * d.vm);
    }

    TileRegs rq, rk, rv;
    float gval = 0.f, gtot = 0.f;
    // The summary pass visits the chunks of its segment in the order opposite to the walk (a sum: each
    // chunk's weights carry the decay of the chunks that follow it in walk order), so that the walker,
    // which runs next, starts with the rows read last.
    auto chunk_of = [&](int kk) { return (REV != SUMMARY) ? kend - 1 - kk : kbeg + kk; };
    auto gload = [&](int kk) {
        const ChunkPos p = walk_pos(d, walk, chunk_of(min(kk, cnt - 1)));
        if (DEC) {
            const int row = min(lane, p.L - 1), tok = REV ? p.L - 1 - row : row;
            gval = a.g[d.kind == 1 ? size_t(walk.bh % d.H) : p.tok0 + size_t(tok) * p.ts];
        }
        if (!SUMMARY) walk_gload<REV, kThreads>(rq, a.xq, p.tok0, p.ts, p.L, tid);
        walk_gload<REV, kThreads>(rk, a.xk, p.tok0, p.ts, p.L, tid);
        walk_gload<REV, kThreads>(rv, a.xv, p.vtok0, p.vts, p.L, tid);
    };
    if (cnt > 0) gload(0);

    for (int kk = 0; kk < cnt; ++kk) {
        const ChunkPos cp = walk_pos(d, walk, chunk_of(kk));
        const int L = cp.L;
        // ---- registers of this chunk -> LDS; decay tables; loads of the next chunk
        if (!SUMMARY) walk_commit<kThreads>(Q, rq, L, tid);
        walk_commit<kThreads>(K, rk, L, tid);
        walk_commit<kThreads>(V, rv, L, tid);
        if (DEC && wave == 0) gtot += walk_decay_tables<REV>(gval, L, SUMMARY ? gtot : 0.f, bs, wo, lane);
        gload(kk + 1);
        __syncthreads();  // (A) tiles and decay tables of this chunk are in LDS
        const float bC = DEC ? bs[C] : 0.f;

        if (!SUMMARY) {
            f32x16 O[2];
            walk_inter<DEC>(O, S, Q, bs, n, half);
            walk_scores<DEC>(K, Q, Ph, Pl, bs, wave, n, half);
            __syncthreads();  // (C) scores are in LDS; nobody reads Q any more
            _Pragma("unroll") for (int jb = 0; jb < 2; ++jb) {
                walk_intra(O[jb], jb, V, Ph, Pl, wave, lane, n, half);
                store_packed(stage, LD, 32 * jb + n, 32 * wave, half, pack_block(O[jb]));
            }
        }
        walk_update<DEC, !SUMMARY>(S, K, V, wo, bC, wave, lane, half);
        __syncthreads();  // (D) the output stage is complete and every read of this chunk's tiles is done
        // every thread reads back exactly the stage pieces that its own next walk_commit overwrites: no barrier
        if (!SUMMARY) walk_store<REV>(a.out, stage, cp.vtok0, cp.vts, L, tid);
    }

    // ---- the state this walk ends with
    if (SUMMARY) {
        const size_t slot = bound_slot(d, walk, a.m, a.nseg) + seg;
        walk_state_store(S, a.bound + (REV ? slot - 1 : slot + 1) * D * D, false, wave, n, half);
        if (tid == 0) a.gseg[slot] = gtot;
        return;
    }
    if (last && a.edge_out) walk_state_store(S, a.edge_out + edge_off(d, walk.edge), false, wave, n, half, D * d.vm);
}

// forward walker, or the summary pass of either direction (grid: segments x sequences; packed input: seg_index)
template <bool REV, bool DEC, bool SUMMARY>
__global__ __launch_bounds__(kThreads, 2) void mk_walk(Dims d, WalkArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SegIndex i = seg_index(d, a.m, blockIdx.x, blockIdx.y);
    if (i.seg < 0) return;
    walk_body<REV, DEC, SUMMARY>(d, a, i.walk, i.seg, smem);
}

// ---------------------------------------------------------------------------------------------
// Gradient walker: dq, dk, dv and the decay gradient of a segment of chunks in one pass, forward in
// time, with the state S (as S^T: rows v, columns i) in accumulators and the state gradients dS read
// from memory, one per chunk (written by the reverse scan, fragment-major bf16).  Per chunk, with
// S = state at the chunk start, dS = gradient of the state at the chunk end, D_jr = e^{b_j-b_r} (r <= j):
//   G = (dO V^T) * D ,  As = (Q K^T) * D
//   dq^T[i][j] = e^{b_j}     sum_v S[i][v]  d_o_j[v] + sum_r K^T[i][r] G[j][r]
//   dk^T[i][r] = e^{b_C-b_r} sum_v dS[i][v] v_r[v]   + sum_j Q^T[i][j] G[j][r]
//   dv^T[v][r] = e^{b_C-b_r} sum_i dS^T[v][i] k_r[i] + sum_j dO^T[v][j] As[j][r]
//   S   <- e^{b_C} S + sum_r e^{b_C-b_r} k_r^T v_r
//   dg_t = sum_{u>=t} (q_u.dq_u - k_u.dk_u) + <S, dS>      (S after the update: the state at the chunk end)
// S enters its product as bf16 head + remainder taken from the fp32 accumulators, so the q.dq term of the decay
// gradient sees no state rounding.  G and As are each computed once per workgroup, one wave per 32 x 32 block, and
// parked as head + remainder in areas of their own; the dS rows, which arrive as the A operands of the dk inter part,
// also go to LDS for the contractions over i.  One workgroup per compute unit, four barriers per chunk
// (VSPLIT: three, its gradients leave from the registers).
// LDS: Q | K | V | dO (64 x LD; at the end the stages of dq, dk, dv) | G head | G remainder | As head |
//      As remainder (64 x LDP each) | dS rows (128 x LD) | bs | wo | red (4 x 2 x 64) | zred
constexpr int kWalkGradLds = (4 * C * LD + 4 * C * LDP + D * LD) * 2 + (2 * C + 8) * 4 + 4 * 64 * 2 * 4 + 64;

struct GradArgs {
    const uint16_t *q, *k, *v, *d_o;
    const float* g;
    const uint16_t* dstates;  // [BH*N] fragment-major bf16: slot c = gradient of the state at the end of chunk c
    uint16_t *dq, *dk, *dv;
    float* dg_tok;            // per-token scalar kind: d_log_decay itself; per-head kind: [BH*N] per-chunk sums
    const float* edge_in;     // M_0 [i][v] per sequence or NULL
    const float* bound;       // entry states of the segments but the first ([i][v]) when nseg > 1
    int m, nseg;
    // VSPLIT: remainder plane of the values (same layout as v); W, the gradient of the delta rule's right-hand side, head and
    // remainder ([BH*T][128] in the library's own order); erase strength per token (NULL = 1) and its gradient (may be NULL)
    const uint16_t *v_lo, *w_h, *w_l;
    const float* beta;
    float* d_beta;
    // the entry states may be kept at a finer grain than this walk's segments: bound is numbered for bound_n segments per sequence,
    // one per m / bound_per chunks, and segment s enters with slot s * bound_per (0: same grain, nseg slots)
    int bound_per, bound_n;
    // d_v = 256 (two passes, one per 128-wide value slice; dq and dk sum over them): the first pass leaves its dq and dk as
    // bf16 head + remainder in these four planes ([BH*T][128], library order: dq head, dq remainder, dk head, dk remainder),
    // the second adds them to its own before the one rounding
    uint16_t* part[4];
};
// VSPLIT (the delta-rule backward, whose values are the pseudo-values U = head + remainder): the values enter every product with
// both planes, the value gradient is not formed (the reverse walk leaves it), and the erase term adds a second set of scores
// and a second query-side gradient (the formulas stand before mk_delta_rwalk):
//   H_tr = -D_tr (W_t . u_r) , r < t ,   X_t = -e^{b_t} S W_t + sum_r H_tr k_r ,   d beta_t = k_t . X_t ,
//   dk_t += beta_t X_t + sum_{j > t} beta_j H_jt k_j ,   dg as for a second query with gradient beta_t X_t.
// The area of As holds beta H; that of the dS rows the two planes of W, then beta X (fp32), which the group that has the rest
// of dk adds before the one rounding.  d beta takes the score part as row sums of H * (K K^T), unscaled (beta may be 0).
// Entry states of the segments come from the forward walk (delta_grad_plan).
constexpr int LDX = 34;  // floats per row of a wave's 64 x 32 part of the stage of beta X
constexpr int kWalkGradSplitExtra = C * LD * 2 + (C + 3 * 32 + 4 * C) * 4;  // second value tile | beta | row sums | k . X per wave
__host__ __device__ constexpr int walk_grad_lds(bool vsplit) { return kWalkGradLds + (vsplit ? kWalkGradSplitExtra : 0); }
static_assert(walk_grad_lds(true) <= 160 * 1024 && C * LDX * 4 <= 32 * LD * 2, "LDS; a wave's beta X fits half of a plane of W");
// a D-layout block whose lanes are tokens (tok, and its row of 128 elements) to memory as bf16, 16 bytes a lane: the halves of a
// wave exchange theirs as in state_store_direct
__device__ __forceinline__ void store_tokens_direct(uint16_t* row, bool ok, int wave, int half, const f32x16& x) {
    const PackedBlock p = pack_block(x);
    _Pragma("unroll") for (int q = 0; q < 2; ++q) {
        const auto s0 = __builtin_amdgcn_permlane32_swap(p.v[2 * q].x, p.v[2 * q + 1].x, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(p.v[2 * q].y, p.v[2 * q + 1].y, false, false);
        if (ok) *reinterpret_cast<u32x4*>(row + 32 * wave + 16 * q + 8 * half) = u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
}

// two inter products with one conversion of the state blocks: X^T[i][t] = sum_v S[i][v] (Wh + Wl)[t][v] (remainder x remainder
// left out) and O^T[i][t] = sum_v S[i][v] Q[t][v]
__device__ __forceinline__ void walk_inter_pair(f32x16 (&X)[2], f32x16 (&O)[2], const f32x16 (&S)[4], const uint16_t* Wh, const uint16_t* Wl,
                                                const uint16_t* Q, int n, int half) {
    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) X[nb] = O[nb] = f32x16{0};
    _Pragma("unroll") for (int ib = 0; ib < 4; ++ib)
        _Pragma("unroll") for (int p = 0; p < 2; ++p) {
            u32x4 hi, lo;
            split_frag(S[ib], p, hi, lo);
            const bf16x8 sh = __builtin_bit_cast(bf16x8, hi), sl = __builtin_bit_cast(bf16x8, lo);
            _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                const bf16x8 wh = frag_perm(Wh, LD, 32 * nb + n, 32 * ib + 16 * p, half);
                const bf16x8 wl = frag_perm(Wl, LD, 32 * nb + n, 32 * ib + 16 * p, half);
                const bf16x8 q = frag_perm(Q, LD, 32 * nb + n, 32 * ib + 16 * p, half);
                X[nb] = mfma(sh, wh, X[nb]);
                O[nb] = mfma(sh, q, O[nb]);
                X[nb] = mfma(sl, wh, X[nb]);
                O[nb] = mfma(sl, q, O[nb]);
                X[nb] = mfma(sh, wl, X[nb]);
            }
        }
}

// score_block2 with rows in two planes: (A + A2)[m] . B[n], and with B2 (A + A2) . (B + B2); the remainders' products apart, so that
// the chains are short.  (The product of two remainders is as large as the rounding of either row: d beta, 16 x 16 sequences of
// 2048, 2-norm 8.1e-6 without it, 7.7e-6; backward 655 and 658 us.)
__device__ __forceinline__ f32x16 score_block_split(const uint16_t* Am, const uint16_t* Am2, int m0, const uint16_t* Bm, const uint16_t* Bm2,
                                                    int n0, int n, int half) {
    f32x16 acc = {0}, rem = {0};
    _Pragma("unroll") for (int h4 = 0; h4 < 2; ++h4) {
        bf16x8 a[4], a2[4], b[4], b2[4];
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
            const int col = 16 * (4 * h4 + ks) + 8 * half;
            a[ks] = frag(Am, LD, m0 + n, col);
            b[ks] = frag(Bm, LD, n0 + n, col);
            a2[ks] = frag(Am2, LD, m0 + n, col);
            if (Bm2) b2[ks] = frag(Bm2, LD, n0 + n, col);
        }
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
            acc = mfma(a[ks], b[ks], acc);
            rem = mfma(a2[ks], b[ks], rem);
            if (Bm2) {
                rem = mfma(a2[ks], b2[ks], rem);
                rem = mfma(a[ks], b2[ks], rem);
            }
        }
    }
    _Pragma("unroll") for (int x = 0; x < 16; ++x) acc[x] += rem[x];
    return acc;
}

// Gradient walker kernel: eight waves, two per SIMD.  The work of a chunk is split by function, not by data, so that
// neither group needs the other's registers:
//   waves 0..3 (wave w: key features i in [32w, 32w+32)) carry the state; they form dq (inter part from the state, intra
//              part from G), <S, dS>, with VSPLIT X, and move the state on;
//   waves 4..7 (wave w: the same i slice for dk, value features v in [32w, 32w+32) for dv) hold the dS rows of the chunk;
//              they compute the score blocks (G, As), dk and dv.
// Each group runs a loop of its own with the same barriers per chunk, so a SIMD always has one wave of either
// kind to issue from: the matrix, vector and LDS work of the two overlap instead of queueing behind one wave's waits.
// Plain case: all 512 threads share the tile traffic (global -> registers -> LDS, stage -> global), and the carrier
// waves read dS for <S, dS> at the (i, v) of their state registers from the LDS rows.
// VSPLIT: the other group moves most of the tiles; the carrier waves form the state's part of X and dq with one conversion of the
// state before barrier (2), then park beta X, complete dq, move the state on and take <S, dS> (dS by loads of their own from the
// fragment-major array, which the other group has just pulled into L2: the LDS area of the dS rows holds W); the other group
// forms the scores before (2) and all of dk, X's scores' share included, after it.  16 x 16 sequences of 2048, 2.8 KB a token: 514 us
// with X completed by the carrier waves and one group moving all tiles but one, 470, 455 with frag_tr4's order, so.
constexpr int kGrad8Threads = 512;

// WIDE: 0 the only pass; 1 the first of two value-slice passes (dq, dk to the partial planes); 2 the second
template <bool DEC, bool WANT_DG, bool VSPLIT = false, int WIDE = 0>
__global__ __launch_bounds__(kGrad8Threads, 1) void mk_walk_grad(Dims d, GradArgs a) {
    static_assert(!(VSPLIT && WIDE), "the two-plane case has 128 value columns");
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* Q = reinterpret_cast<uint16_t*>(smem);
    uint16_t* K = Q + C * LD;
    uint16_t* V = K + C * LD;
    uint16_t* dO = V + C * LD;
    uint16_t* Gh = dO + C * LD;
    uint16_t* Gl = Gh + C * LDP;
    uint16_t* Ah = Gl + C * LDP;
    uint16_t* Al = Ah + C * LDP;
    uint16_t* dSt = Al + C * LDP;    // [i][v] rows of dS, all 128
    float* bs = reinterpret_cast<float*>(dSt + D * LD);
    float* wo = bs + C + 4;
    float* red = wo + C + 4;         // [i slice][2][64]: q.dq, k.dk partial sums over the slice
    float* zred = red + 4 * 2 * 64;  // [i slice]: partial <S, dS>
    uint16_t* V2 = reinterpret_cast<uint16_t*>(smem + kWalkGradLds);  // VSPLIT only
    uint16_t* Wh = dSt;              // VSPLIT: 64 x LD each, over the dS rows
    uint16_t* Wl = dSt + C * LD;
    // ... and, once they are spent, beta X: a wave's [64][LDX] over the rows of W that the wave of the same index among the others
    // writes next
    float* Xs = reinterpret_cast<float*>(dSt) + (int(threadIdx.x >> 6) & 3) * (32 * LD / 2);
    float* be = reinterpret_cast<float*>(smem + kWalkGradLds + C * LD * 2);  // VSPLIT: beta [64]
    float* rowF = be + C;            // [block][32]: sum_r H_tr (k_t . k_r) over the block's keys
    float* redx = rowF + 3 * 32;     // [i slice][64]: k . X without the scores' share
    uint16_t* Lq = Gh;               // WIDE == 1: stages of the remainder planes of dq and dk (G and As are spent after (3))
    uint16_t* Lk = Ah;
    static_assert(2 * C * LDP >= C * LD, "a 64 x LD stage fits the area of G");
    constexpr int NT = VSPLIT ? 256 : kGrad8Threads;  // threads that share the tile traffic

    const SegIndex si = seg_index(d, a.m, blockIdx.x, blockIdx.y);
    if (si.seg < 0) return;
    const SeqWalk walk = si.walk;
    const int seq = walk.edge, seg = si.seg;
    // the wave index as a scalar: the branch between the two groups is then a scalar branch (each group's barriers are
    // executed by its own waves only, whatever the compiler makes of the vector condition), and 32 * wave offsets are scalars
    const int tid = threadIdx.x, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3;
    int lane = tid & 63, n = lane & 31, half = lane >> 5;
    int tt = VSPLIT ? tid & 255 : tid;  // index among the threads that move tiles
    const bool carrier = wave8 < 4;     // waves 0..3
    // VSPLIT: every LDS access pattern keeps a lane-dependent base address per 64 KiB window of the 159 KiB
    // in use, and with the state, two sets of accumulators and the tiles in flight there is no room to keep a hundred of
    // them alive across the loop.  Hiding the lane id from the optimiser at the phase boundaries makes it recompute the
    // addresses of a phase inside the phase (a few vector instructions each) instead of spilling them.
    auto fresh = [&]() {
        if (VSPLIT) {
            asm volatile("" : "+v"(lane));
            n = lane & 31;
            half = lane >> 5;
            tt = 64 * wave + lane;
        }
    };
    const int kbeg = seg * a.m, kend = min(walk.n, kbeg + a.m), cnt = kend - kbeg;
    if (cnt <= 0) return;

    // VSPLIT: the carrier group moves q, k and d_o in, the other group the planes of U and W; the gradients leave from the
    // registers.  Requests are made after (2), under the products.  (One group moving all but a tile, between the chunks: 2300 clocks
    // to issue, 2200 to commit, of 24500.)
    // Wave w of the other group moves rows 32 (w % 2) .. + 31 of the head (w < 2) or remainder plane of W.
    TileRegs tq, tk, tv, to, tv2;
    u32x4 tw[8];
    auto gload_tiles = [&](const ChunkPos& p, bool first_group) {
        if (!VSPLIT || first_group) {
            walk_gload<false, NT>(tq, a.q, p.tok0, p.ts, p.L, tt);
            walk_gload<false, NT>(tk, a.k, p.tok0, p.ts, p.L, tt);
        }
        if (!VSPLIT || !first_group) walk_gload<false, NT>(tv, a.v, p.vtok0, p.vts, p.L, tt);
        if (!VSPLIT || first_group) walk_gload<false, NT>(to, a.d_o, p.vtok0, p.vts, p.L, tt);
        if (VSPLIT && !first_group) {
            walk_gload<false, NT>(tv2, a.v_lo, p.vtok0, p.vts, p.L, tt);
            const uint16_t* w = (wave < 2 ? a.w_h : a.w_l) + p.wtok0 * D;
            _Pragma("unroll") for (int it = 0; it < 8; ++it)
                tw[it] = *reinterpret_cast<const u32x4*>(w + min(32 * (wave & 1) + 4 * it + (lane >> 4), p.L - 1) * D + 8 * (lane & 15));
        }
    };
    auto commit_tiles = [&](int L, bool first_group) {
        if (VSPLIT && !first_group) {
            _Pragma("unroll") for (int it = 0; it < 8; ++it) {
                const int row = 32 * (wave & 1) + 4 * it + (lane >> 4);
                const uint32_t keep = row < L ? 0xffffffffu : 0u;
                *reinterpret_cast<u32x4*>((wave < 2 ? Wh : Wl) + row * LD + 8 * (lane & 15)) =
                    u32x4{tw[it].x & keep, tw[it].y & keep, tw[it].z & keep, tw[it].w & keep};
            }
        }
        if (!VSPLIT || first_group) {
            walk_commit<NT>(Q, tq, L, tt);
            walk_commit<NT>(K, tk, L, tt);
        }
        if (!VSPLIT || !first_group) walk_commit<NT>(V, tv, L, tt);
        if (!VSPLIT || first_group) walk_commit<NT>(dO, to, L, tt);
        if (VSPLIT && !first_group) walk_commit<NT>(V2, tv2, L, tt);
    };
    auto store_tiles = [&](const ChunkPos& cp) {
        // Every thread reads back exactly the stage pieces that its own next commit overwrites: no barrier between this and
        // the next chunk's commit.
        if (WIDE == 1) {  // head and remainder of this pass's dq and dk, for the second pass
            walk_store<false, NT>(a.part[0], Q, cp.wtok0, 1, cp.L, tt);
            walk_store<false, NT>(a.part[1], Lq, cp.wtok0, 1, cp.L, tt);
            walk_store<false, NT>(a.part[2], K, cp.wtok0, 1, cp.L, tt);
            walk_store<false, NT>(a.part[3], Lk, cp.wtok0, 1, cp.L, tt);
        } else {
            walk_store<false, NT>(a.dq, Q, cp.tok0, cp.ts, cp.L, tt);
            walk_store<false, NT>(a.dk, K, cp.tok0, cp.ts, cp.L, tt);
        }
        walk_store<false, NT>(a.dv, V, cp.vtok0, cp.vts, cp.L, tt);
    };
    // WIDE == 2: the first pass's share of a gradient block (lane = token 32 nb + n, registers = this wave's 32 features)
    struct Part { u32x2 h[4], l[4]; };
    auto part_load = [&](Part& pt, const uint16_t* ph, const uint16_t* pl, const ChunkPos& cp, int nb) {
        const size_t row = (cp.wtok0 + size_t(min(32 * nb + n, max(cp.L, 1) - 1))) * D + 32 * wave + 4 * half;
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            pt.h[g] = *reinterpret_cast<const u32x2*>(ph + row + 8 * g);
            pt.l[g] = *reinterpret_cast<const u32x2*>(pl + row + 8 * g);
        }
    };
    auto part_add = [](f32x16& x, const Part& pt) {
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            x[4 * g + 0] += bf16_lo(pt.h[g].x) + bf16_lo(pt.l[g].x);
            x[4 * g + 1] += bf16_hi(pt.h[g].x) + bf16_hi(pt.l[g].x);
            x[4 * g + 2] += bf16_lo(pt.h[g].y) + bf16_lo(pt.l[g].y);
            x[4 * g + 3] += bf16_hi(pt.h[g].y) + bf16_hi(pt.l[g].y);
        }
    };
    // head of a block; the block keeps its remainder
    auto split_block = [](f32x16& x) {
        const PackedBlock h = pack_block(x);
        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
            x[4 * g + 0] -= bf16_lo(h.v[g].x);
            x[4 * g + 1] -= bf16_hi(h.v[g].x);
            x[4 * g + 2] -= bf16_lo(h.v[g].y);
            x[4 * g + 3] -= bf16_hi(h.v[g].y);
        }
        return h;
    };

    if (carrier) {
        // S block vb of this wave: S[vb][4g+j] = M[i = 32 wave + n][v = 32 vb + 8g + 4 half + j]
        f32x16 S[4];
        _Pragma("unroll") for (int vb = 0; vb < 4; ++vb) S[vb] = f32x16{0};
        {
            const int per = a.bound_per ? a.bound_per : 1;
            if (seg > 0)
                walk_state_load(S, a.bound + (bound_slot(d, walk, a.m / per, a.bound_per ? a.bound_n : a.nseg) + seg * per) * D * D, true, wave, n, half);
            else if (a.edge_in) walk_state_load(S, a.edge_in + edge_off(d, seq), true, wave, n, half, D * d.vm);
        }
        float gval = 0.f, bval = 1.f;
        auto gload = [&](int kk) {
            const ChunkPos p = walk_pos(d, walk, kbeg + min(kk, cnt - 1));
            if (VSPLIT && a.beta) bval = a.beta[p.tok0 + size_t(min(lane, p.L - 1)) * p.ts];
            if (DEC) gval = a.g[d.kind == 1 ? size_t(walk.bh % d.H) : p.tok0 + size_t(min(lane, p.L - 1)) * p.ts];
            gload_tiles(p, true);
        };
        // dq^T[i][j] += sum_{r<=j} K^T[i][r] G[j][r] (keys r >= 32 never reach queries j < 32), its share of the decay gradient
        auto dq_intra = [&](f32x16 (&aq)[2], PackedBlock (&resq)[2], PackedBlock (&resql)[2], const ChunkPos& cp) {
            Part pt[2];
            if (WIDE == 2) {
                part_load(pt[0], a.part[0], a.part[1], cp, 0);
                part_load(pt[1], a.part[0], a.part[1], cp, 1);
            }
            _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                const int tok = 32 * nb + n;
                _Pragma("unroll") for (int ks = 0; ks < 2 * (nb + 1); ++ks) {
                    const bf16x8 kt = frag_tr(K, LD, 16 * ks, 32 * wave, lane);
                    aq[nb] = mfma(kt, frag(Gh, LDP, tok, 16 * ks + 8 * half), aq[nb]);
                    aq[nb] = mfma(kt, frag(Gl, LDP, tok, 16 * ks + 8 * half), aq[nb]);
                }
                if (WANT_DG) {
                    float pq = row_dot(Q, tok, wave, half, aq[nb]);
                    pq += __shfl_xor(pq, 32, 64);
                    if (half == 0) red[(wave * 2 + 0) * 64 + tok] = pq;
                }
                if (WIDE == 2) part_add(aq[nb], pt[nb]);  // after the decay gradient took this pass's own share
                if (WIDE == 1) {
                    resq[nb] = split_block(aq[nb]);
                    resql[nb] = pack_block(aq[nb]);
                } else {
                    resq[nb] = pack_block(aq[nb]);
                }
            }
        };
        // <S, dS> with the state at the END of the chunk, over this wave's rows i: together with the running sums of
        // q.dq - k.dk this is the whole decay gradient (<e^{b_C} S + S_chunk, dS> = e^{b_C} <S, dS> + sum_r k_r.dk_r^{inter}).
        // dS at the (i, v) of the state registers: from the LDS rows, or (VSPLIT) from the registers dsz
        auto state_dot = [&](const u32x2 (&dsz)[16]) {
            float z = 0.f;
            _Pragma("unroll") for (int vb = 0; vb < 4; ++vb)
                _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                    const u32x2 x = VSPLIT ? dsz[4 * vb + g]
                                           : *reinterpret_cast<const u32x2*>(dSt + (32 * wave + n) * LD + 32 * vb + 8 * g + 4 * half);
                    z += S[vb][4 * g] * bf16_lo(x.x) + S[vb][4 * g + 1] * bf16_hi(x.x) + S[vb][4 * g + 2] * bf16_lo(x.y) +
                         S[vb][4 * g + 3] * bf16_hi(x.y);
                }
            for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off, 64);
            if (lane == 0) zred[wave] = z;
        };
        gload(0);
        for (int kk = 0; kk < cnt; ++kk) {
            const ChunkPos cp = walk_pos(d, walk, kbeg + kk);
            const int L = cp.L;
            fresh();
            commit_tiles(L, true);
            if (DEC && wave8 == 0) walk_decay_tables<false>(gval, L, 0.f, bs, wo, lane);
            if (VSPLIT && wave8 == 0) be[lane] = lane < L ? bval : 0.f;
            __syncthreads();  // (1) tiles, dS rows and decay tables of this chunk are in LDS
            fresh();
            const float bC = DEC ? bs[C] : 0.f;
            f32x16 aq[2], ax[2];
            PackedBlock resq[2], resql[2];
            if (VSPLIT) {
                // X^T[i][t] and dq^T[i][t], the state's share: -e^{b_t} sum_v S[i][v] W[t][v], e^{b_t} sum_v S[i][v] dO[t][v]
                walk_inter_pair(ax, aq, S, Wh, Wl, dO, n, half);
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    const int tok = 32 * nb + n;
                    const float w = DEC ? __expf(bs[tok]) : 1.f, b = be[tok];
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) {
                        if (DEC) aq[nb][x] *= w;
                        ax[nb][x] *= -w;
                    }
                    float px = row_dot(K, tok, wave, half, ax[nb]);
                    px += __shfl_xor(px, 32, 64);
                    if (half == 0) redx[wave * 64 + tok] = px;
                    _Pragma("unroll") for (int x = 0; x < 16; ++x) ax[nb][x] *= b;
                }
            } else {
                walk_inter<DEC>(aq, S, dO, bs, n, half);
            }
            u32x2 dsz[16];  // VSPLIT: dS at the (i, v) of the state registers, four consecutive v per load
            if (!VSPLIT) {
                // the state moves on to the end of the chunk (roles: key = v, value = k)
                walk_update<DEC, true>(S, V, K, wo, bC, wave, lane, half);
                if (WANT_DG) state_dot(dsz);
                if (kk + 1 < cnt) gload(kk + 1);
            }
            __syncthreads();  // (2) G and As are in LDS
            fresh();
            if (VSPLIT) {
                // (a chain of few products: every operand is requested before anything is written to LDS)
                bf16x8 kt[4], gh[6], gl[6];
                _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) kt[ks] = frag_tr(K, LD, 16 * ks, 32 * wave, lane);
                _Pragma("unroll") for (int i = 0; i < 6; ++i) {
                    const int off = (i < 2 ? n : 32 + n) * LDP + 16 * (i < 2 ? i : i - 2) + 8 * half;
                    gh[i] = *reinterpret_cast<const bf16x8*>(Gh + off);
                    gl[i] = *reinterpret_cast<const bf16x8*>(Gl + off);
                }
                _Pragma("unroll") for (int i = 0; i < 6; ++i) {
                    aq[i < 2 ? 0 : 1] = mfma(kt[i < 2 ? i : i - 2], gl[i], aq[i < 2 ? 0 : 1]);
                    aq[i < 2 ? 0 : 1] = mfma(kt[i < 2 ? i : i - 2], gh[i], aq[i < 2 ? 0 : 1]);
                }
                if (WANT_DG) {
                    float pq[2];
                    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) pq[nb] = row_dot(Q, 32 * nb + n, wave, half, aq[nb]);
                    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                        pq[nb] += __shfl_xor(pq[nb], 32, 64);
                        if (half == 0) red[(wave * 2 + 0) * 64 + 32 * nb + n] = pq[nb];
                    }
                }
                // the planes of W are spent: beta X (without the scores' share) is parked over them for the group that has dk
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb)
                    _Pragma("unroll") for (int g = 0; g < 4; ++g)
                        _Pragma("unroll") for (int h = 0; h < 2; ++h)
                            *reinterpret_cast<float2*>(Xs + (32 * nb + n) * LDX + 8 * g + 4 * half + 2 * h) = float2{ax[nb][4 * g + 2 * h], ax[nb][4 * g + 2 * h + 1]};
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb)
                    store_tokens_direct(a.dq + (cp.tok0 + size_t(32 * nb + n) * cp.ts) * D, 32 * nb + n < L, wave, half, aq[nb]);
                if (kk + 1 < cnt) gload(kk + 1);
                fresh();
                if (WANT_DG) {
                    const uint16_t* dS = a.dstates + cp.slot * D * D;
                    _Pragma("unroll") for (int vb = 0; vb < 4; ++vb)
                        _Pragma("unroll") for (int g = 0; g < 4; ++g)
                            dsz[4 * vb + g] = *reinterpret_cast<const u32x2*>(dS + state_frag_off(wave, 2 * vb + (g >> 1), 32 * (g & 1) + n) + 4 * half);
                }
                walk_update<DEC, true, true>(S, V, K, wo, bC, wave, lane, half, V2);
                if (WANT_DG) state_dot(dsz);
            } else {
                dq_intra(aq, resq, resql, cp);
            }
            __syncthreads();  // (3) every wave is done with the tiles
            fresh();
            if (!VSPLIT) {
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    store_packed(Q, LD, 32 * nb + n, 32 * wave, half, resq[nb]);
                    if (WIDE == 1) store_packed(Lq, LD, 32 * nb + n, 32 * wave, half, resql[nb]);
                }
                __syncthreads();  // (4)
                store_tiles(cp);
            }
            auto kx = [&]() {  // k_t . X_t; row sums of the scores' share: t < 32 from block (0,0); t >= 32 from (1,0) and (1,1)
                return (redx[lane] + redx[64 + lane]) + (redx[128 + lane] + redx[192 + lane]) + (lane < 32 ? rowF[lane] : rowF[lane] + rowF[32 + lane]);
            };
            if (VSPLIT && a.d_beta && wave8 == 1 && lane < L) a.d_beta[cp.tok0 + size_t(lane) * cp.ts] = kx();
            if (WANT_DG && wave8 == 0) {
                // fixed-order sums over the four feature slices, then the reverse in-chunk running sum
                float w = 0.f;
                const float z = (zred[0] + zred[1]) + (zred[2] + zred[3]);
                _Pragma("unroll") for (int wv = 0; wv < 4; ++wv) w += red[(wv * 2 + 0) * 64 + tid] - red[(wv * 2 + 1) * 64 + tid];
                if (VSPLIT) w += be[tid] * kx();
                float sfx = w;  // suffix sum of w over tokens >= tid
                for (int off = 1; off < 64; off <<= 1) {
                    const float y = __shfl_down(sfx, off, 64);
                    if (tid + off < 64) sfx += y;
                }
                float dgv = tid < L ? sfx + z : 0.f;
                constexpr bool add = WIDE == 2;  // the decay gradient sums over the value slices too
                if (d.kind == 1) {
                    // one decay per head: only the sum over tokens is wanted; this chunk's share, in a fixed order
                    for (int off = 32; off > 0; off >>= 1) dgv += __shfl_xor(dgv, off, 64);
                    if (tid == 0) a.dg_tok[cp.slot] = add ? a.dg_tok[cp.slot] + dgv : dgv;
                } else if (tid < L) {
                    float* pg = a.dg_tok + cp.tok0 + size_t(tid) * cp.ts;
                    *pg = add ? *pg + dgv : dgv;
                }
            }
        }
    } else {
        bf16x8 dsfrag[8];
        auto gload = [&](int kk) {
            const ChunkPos p = walk_pos(d, walk, kbeg + min(kk, cnt - 1));
            if (!VSPLIT) gload_tiles(p, false);
            // rows i in [32w, 32w+32) of dS: A operands [m = i][k = v]
            const uint16_t* dS = a.dstates + p.slot * D * D;
            _Pragma("unroll") for (int ks = 0; ks < 8; ++ks)
                dsfrag[ks] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(dS + state_frag_off(wave, ks, lane)));
        };
        // one 32 x 32 score block (0: (0,0), 1: (1,0), 2: (1,1)), mask and decay on its accumulators, as head + remainder
        auto score = [&](bool isG, int bi) {
            const int pjb = bi ? 1 : 0, prb = bi == 2 ? 1 : 0;
            // D[m = r][n = j] = v_r . d_o_j  or  k_r . q_j
            f32x16 P = !isG ? score_block2(K, 32 * prb, Q, 32 * pjb, n, half)
                       : VSPLIT ? score_block_split(V, V2, 32 * prb, dO, nullptr, 32 * pjb, n, half)
                                : score_block2(V, 32 * prb, dO, 32 * pjb, n, half);
            walk_mask<DEC>(P, 32 * prb, 32 * pjb + n, bs, half);
            store_block_t_split(isG ? Gh : Ah, isG ? Gl : Al, LDP, 32 * pjb + n, 32 * prb, half, P);
        };
        // VSPLIT: a block of H, with its row sums against K K^T; what is kept is beta H
        auto erase_score = [&](int bi) {
            const int pjb = bi ? 1 : 0, prb = bi == 2 ? 1 : 0, t = 32 * pjb + n;
            f32x16 P = score_block_split(V, V2, 32 * prb, Wh, Wl, 32 * pjb, n, half);  // D[m = r][n = t] = u_r . W_t
            walk_mask<DEC>(P, 32 * prb, t, bs, half);
            const f32x16 G = score_block2(K, 32 * prb, K, 32 * pjb, n, half);
            const float b = be[t];
            float rs = 0.f;
            _Pragma("unroll") for (int x = 0; x < 16; ++x) {
                P[x] = 32 * prb + 8 * (x >> 2) + 4 * half + (x & 3) == t ? 0.f : -P[x];  // a key does not erase itself
                rs += P[x] * G[x];
                P[x] *= b;
            }
            rs += __shfl_xor(rs, 32, 64);
            if (half == 0) rowF[32 * bi + n] = rs;
            store_block_t_split(Ah, Al, LDP, t, 32 * prb, half, P);
        };
        if (VSPLIT) gload_tiles(walk_pos(d, walk, kbeg), false);
        gload(0);
        for (int kk = 0; kk < cnt; ++kk) {
            const ChunkPos cp = walk_pos(d, walk, kbeg + kk);
            const int L = cp.L;
            fresh();
            commit_tiles(L, false);
            if (!VSPLIT) {
                // the dS rows of this wave, for the contractions over i (dv, <S, dS>)
                _Pragma("unroll") for (int ks = 0; ks < 8; ++ks)
                    *reinterpret_cast<bf16x8*>(dSt + (32 * wave + n) * LD + 16 * ks + 8 * half) = dsfrag[ks];
            }
            __syncthreads();  // (1)
            fresh();
            // G = (dO V^T) * D first (the other group waits for it at (2)), then As = (Q K^T) * D, which only dv needs
            if (VSPLIT) {
                if (wave < 3) {
                    if (kk + 1 < cnt) gload_tiles(walk_pos(d, walk, kbeg + kk + 1), false);
                    erase_score(wave);
                } else {
                    _Pragma("unroll 1") for (int bi = 0; bi < 3; ++bi) score(true, bi);
                }
            } else {
                if (wave < 3) score(true, wave);
                else score(false, 0);
                if (wave < 2) score(false, wave + 1);
            }
            // inter parts: dk^T[i][r] from the dS rows in registers, dv^T[v][r] from the transposed read of the LDS rows
            f32x16 ak[2] = {{0}, {0}}, av[2] = {{0}, {0}};
            auto dk_inter = [&]() {
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    const int tok = 32 * nb + n;
                    _Pragma("unroll") for (int ks = 0; ks < 8; ++ks) ak[nb] = mfma(dsfrag[ks], frag(V, LD, tok, 16 * ks + 8 * half), ak[nb]);
                    if (VSPLIT) {
                        _Pragma("unroll") for (int ks = 0; ks < 8; ++ks) ak[nb] = mfma(dsfrag[ks], frag(V2, LD, tok, 16 * ks + 8 * half), ak[nb]);
                    }
                    if (DEC) {
                        const float wk = wo[tr4_at(tok)];
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) ak[nb][x] *= wk;
                    }
                }
                if (kk + 1 < cnt) gload(kk + 1);  // the dS registers are free
            };
            if (!VSPLIT) dk_inter();
            if (!VSPLIT) {
                _Pragma("unroll") for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 dst = frag_tr(dSt, LD, 16 * ks, 32 * wave, lane);  // dS^T[v][i], i = 16 ks + ..
                    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb)
                        av[nb] = mfma(dst, frag(K, LD, 32 * nb + n, 16 * ks + 8 * half), av[nb]);
                }
                if (DEC) {
                    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                        const float wk = wo[tr4_at(32 * nb + n)];
                        _Pragma("unroll") for (int x = 0; x < 16; ++x) av[nb][x] *= wk;
                    }
                }
            }
            __syncthreads();  // (2) G and As are in LDS
            fresh();
            if (VSPLIT) {
                if (wave == 3 && kk + 1 < cnt) gload_tiles(walk_pos(d, walk, kbeg + kk + 1), false);
                dk_inter();
            }
            PackedBlock resk[2], resv[2], reskl[2];
            Part pt[2];
            if (WIDE == 2) {
                part_load(pt[0], a.part[2], a.part[3], cp, 0);
                part_load(pt[1], a.part[2], a.part[3], cp, 1);
            }
            if (VSPLIT) {
                // dk^T[i][r] += sum_{j>=r} Q^T[i][j] G[j][r], the same with beta H and the keys in the query's place, then, after the
                // decay gradient took the key side, the scores' share of beta X.  Remainders and far queries first, the token's own
                // query, the largest term under a decay, last: q.dq and k.dk share it and the decay gradient is what is left of the
                // two, so that what is added after it would be rounded at its size (d log alpha, decays of e^-4, 2-norm 2.05e-5 the
                // other way round, 1.89e-5 so).
                bf16x8 qt[4], kt[4];
                _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {
                    qt[ks] = frag_tr4(Q, LD, 16 * ks, 32 * wave, lane);
                    kt[ks] = frag_tr4(K, LD, 16 * ks, 32 * wave, lane);
                }
                float pk[2] = {0.f, 0.f};
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    _Pragma("unroll") for (int ks = 3; ks >= 2 * nb; --ks) {
                        ak[nb] = mfma(kt[ks], frag_tr4(Al, LDP, 16 * ks, 32 * nb, lane), ak[nb]);
                        ak[nb] = mfma(kt[ks], frag_tr4(Ah, LDP, 16 * ks, 32 * nb, lane), ak[nb]);
                        ak[nb] = mfma(qt[ks], frag_tr4(Gl, LDP, 16 * ks, 32 * nb, lane), ak[nb]);
                        ak[nb] = mfma(qt[ks], frag_tr4(Gh, LDP, 16 * ks, 32 * nb, lane), ak[nb]);
                    }
                    if (WANT_DG) pk[nb] = row_dot(K, 32 * nb + n, wave, half, ak[nb]);
                    _Pragma("unroll") for (int ks = 0; ks < 2 * (nb + 1); ++ks) {
                        const bf16x8 kn = frag_tr(K, LD, 16 * ks, 32 * wave, lane);
                        ak[nb] = mfma(kn, frag(Ah, LDP, 32 * nb + n, 16 * ks + 8 * half), ak[nb]);
                        ak[nb] = mfma(kn, frag(Al, LDP, 32 * nb + n, 16 * ks + 8 * half), ak[nb]);
                    }
                }
                if (WANT_DG) {
                    _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                        pk[nb] += __shfl_xor(pk[nb], 32, 64);
                        if (half == 0) red[(wave * 2 + 1) * 64 + 32 * nb + n] = pk[nb];
                    }
                }
            }
            _Pragma("unroll") for (int nb = 0; nb < (VSPLIT ? 0 : 2); ++nb) {
                const int tok = 32 * nb + n;
                // dk^T[i][r] += sum_{j>=r} Q^T[i][j] G[j][r]: queries j < 32 never see keys r >= 32
                _Pragma("unroll") for (int ks = 2 * nb; ks < 4; ++ks) {
                    const bf16x8 qt = frag_tr(Q, LD, 16 * ks, 32 * wave, lane);
                    ak[nb] = mfma(qt, frag_tr(Gh, LDP, 16 * ks, 32 * nb, lane), ak[nb]);  // B[k = j][n = r] = G[j][r]
                    ak[nb] = mfma(qt, frag_tr(Gl, LDP, 16 * ks, 32 * nb, lane), ak[nb]);
                }
                if (WANT_DG) {
                    float pk = row_dot(K, tok, wave, half, ak[nb]);
                    pk += __shfl_xor(pk, 32, 64);
                    if (half == 0) red[(wave * 2 + 1) * 64 + tok] = pk;
                }
                if (WIDE == 2) part_add(ak[nb], pt[nb]);
                if (WIDE == 1) {
                    resk[nb] = split_block(ak[nb]);
                    reskl[nb] = pack_block(ak[nb]);
                } else {
                    resk[nb] = pack_block(ak[nb]);
                }
                // dv^T[v][r] += sum_{j>=r} dO^T[v][j] As[j][r]
                _Pragma("unroll") for (int ks = 2 * nb; ks < 4; ++ks) {
                    const bf16x8 dot = frag_tr(dO, LD, 16 * ks, 32 * wave, lane);
                    av[nb] = mfma(dot, frag_tr(Ah, LDP, 16 * ks, 32 * nb, lane), av[nb]);  // B[k = j][n = r] = As[j][r]
                    av[nb] = mfma(dot, frag_tr(Al, LDP, 16 * ks, 32 * nb, lane), av[nb]);
                }
                resv[nb] = pack_block(av[nb]);
            }
            __syncthreads();  // (3)
            fresh();
            if (VSPLIT) {  // with the other group's beta X, before the one rounding (the wave's own next rows of W come over it)
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    const int tok = 32 * nb + n;
                    _Pragma("unroll") for (int g = 0; g < 4; ++g)
                        _Pragma("unroll") for (int h = 0; h < 2; ++h) {
                            const float2 x = *reinterpret_cast<const float2*>(Xs + tok * LDX + 8 * g + 4 * half + 2 * h);
                            ak[nb][4 * g + 2 * h] += x.x;
                            ak[nb][4 * g + 2 * h + 1] += x.y;
                        }
                    store_tokens_direct(a.dk + (cp.tok0 + size_t(tok) * cp.ts) * D, tok < L, wave, half, ak[nb]);
                }
            } else {
                _Pragma("unroll") for (int nb = 0; nb < 2; ++nb) {
                    store_packed(K, LD, 32 * nb + n, 32 * wave, half, resk[nb]);
                    store_packed(V, LD, 32 * nb + n, 32 * wave, half, resv[nb]);
                    if (WIDE == 1) store_packed(Lk, LD, 32 * nb + n, 32 * wave, half, reskl[nb]);
                }
                __syncthreads();  // (4)
                store_tiles(cp);
            }
        }
    }
}

// Entry state of every segment from the segments' own contributions (left by the summary pass in the
// slot of the segment that follows in walk order) and total log-decays: E' = e^{G} E + U, in walk order.
// The contributions are read a batch of segments at a time before any of them is replaced: the reads of a batch do not
// depend on each other, only the recurrence does (read - update - write in turn pays one memory latency per segment).
// Eight at a time; MANY: 24 while there are that many left, which holds more registers (many_at_once).
// grid: (128 * 128 / 256, seqs)
template <bool REV, bool MANY>
__global__ __launch_bounds__(kThreads) void mk_bound_scan(Dims d, const float* __restrict__ edge_in, float* __restrict__ bound,
                                                          const float* __restrict__ gseg, int m, int nseg, int skip) {
    const int seq = blockIdx.y, e = blockIdx.x * kThreads + threadIdx.x;
    const SeqWalk walk = seq_walk(d, seq);
    const int nsq = (walk.n + m - 1) / m;
    if (nsq <= 1 && (!REV || nsq == 0)) return;  // forward, the first segment starts from edge_in itself
    const size_t slot = bound_slot(d, walk, m, nseg);
    float* b = bound + slot * D * D + e;
    const float* gs = gseg + slot;
    float E = edge_in ? edge_in[edge_off(d, seq) + size_t(e / D) * D * d.vm + e % D] : 0.f;
    auto batch = [&](auto size, int s0) {
        constexpr int G = decltype(size)::value;
        float u[G], w[G];
        if (!REV) {
            _Pragma("unroll") for (int i = 0; i < G; ++i) {
                const int s = min(s0 + i, nsq - 2);
                u[i] = b[size_t(s + 1) * D * D];
                w[i] = gs[s];
            }
            _Pragma("unroll") for (int i = 0; i < G; ++i)
                if (s0 + i + 1 < nsq) {
                    E = __expf(w[i]) * E + u[i];
                    b[size_t(s0 + i + 1) * D * D] = E;
                }
            return s0 + G;
        } else {
            _Pragma("unroll") for (int i = 0; i < G; ++i) {
                const int s = max(s0 - i, skip);
                u[i] = b[size_t(s - 1) * D * D];
                w[i] = gs[s];
            }
            _Pragma("unroll") for (int i = 0; i < G; ++i)
                if (s0 - i >= skip) {
                    E = __expf(w[i]) * E + u[i];
                    b[size_t(s0 - i - 1) * D * D] = E;
                }
            return s0 - G;
        }
    };
    if (!REV) {
        int s0 = 0;
        if constexpr (MANY)
            while (nsq - 1 - s0 >= 24) s0 = batch(std::integral_constant<int, 24>{}, s0);
        while (s0 + 1 < nsq) s0 = batch(std::integral_constant<int, 8>{}, s0);
    } else {
        b[size_t(nsq - 1) * D * D] = E;
        int s0 = nsq - 1;  // slots below skip - 1 are entered by no walk
        if constexpr (MANY)
            while (s0 - skip + 1 >= 24) s0 = batch(std::integral_constant<int, 24>{}, s0);
        while (s0 >= skip) s0 = batch(std::integral_constant<int, 8>{}, s0);
    }
}
