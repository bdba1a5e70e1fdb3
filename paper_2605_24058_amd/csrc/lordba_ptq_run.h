// The sweeps of a quantisation run as ONE launch (carrier rank up to 16, factor rank up to 32).
//
// A sweep is a chain of four steps - Tikhonov step and duals of U1, the same of U2, alpha, gamma - each of which needs the Gram
// pair of all rows of the side before it.  As launches of their own the steps of 4096^2, R = 16 took 57 us per sweep, of which
// the arithmetic is a fraction, and a run that ends after 22 of its 100 sweeps paid 0.5 ms for the launches behind its end.
// Here the blocks of all steps of all sweeps are numbered in order, and every workgroup takes the next number that nobody has
// taken (one counter), waits until the step before is complete, does the block, publishes its share of the Gram pair and goes on.  A block
// waits for blocks with smaller numbers only, and whoever holds a number does it before any other that it holds, so the smallest unfinished
// one is always being worked on: the launch ends whatever the number of workgroups that run at a time, also beside other work on the
// device, and none of them has to be there.  (No result depends on who does which block; sums run in a fixed order.)
//
// What one workgroup writes and another reads goes through agent-scope accesses (see `publish`).  Two kinds of waiting:
//   - For the shares of the step before, which is all that the chain of steps hangs on, by the shares themselves: each value carries the
//     parity of its sweep in a bit of its exponent (with_mark), and a reader takes the shares as they come.  That needs no wait for the stores, no
//     arrival and no second trip to memory behind it: 2 us of a step's 12.  What lay in a share's place before has to be known: the first
//     sweep of a launch goes by the arrivals, and before a reader looks at the shares of sweep t it has seen an arrival that implies that
//     those of sweep t - 1 are complete (or it could find those of t - 2, which carry the same mark).
//   - For rows, scales, gaps and beta by arrival counters, one per kind of step; a workgroup counts itself when every wave's stores have
//     completed (see `arrive_last`).  These waits come early in a block: what they are for was written a step or more before.
// Buffers that a later step overwrites have no reader left by then: a step publishes when it has read all shares of the step before, and
// readers are at most three steps behind their writer; what is read longer (beta, penalty, consensus gaps) is kept twice, by the parity of
// the sweep.
//
// Time of a sweep of 4096^2, R = r0 = 16 (64 and 32 workgroups): 38 us, 48 with arrivals for everything, a number asked for when the block
// before is done (64 workgroups queue 7 us for it) and the loads of a scale step one behind the other.  U1's step 11.8 (shares on their way
// 1.2, added up 2, beta 3.9, rows 5, share 0.7), U2's 10.5, alpha 8, gamma 6; bound: the chain, in it 64-bit vector arithmetic of four waves
// per SIMD (rows) and 64 bytes per clock into a compute unit (shares: 64 of 3136 bytes).
//
// Blocks: 64 rows of a Tikhonov step (16 waves, four rows each; a lane group per row as in row_ldlt_solve), 128 rows of a
// scale step (8 of the waves, 16 rows each), more per block beyond 4096 or 8192 rows, so that a step has at most 64 blocks whose
// shares every reader adds up.  Fewer rows per scale block give readers more shares, more put the 64-bit MFMAs of four waves behind each
// other (ms per call, R = r0 = 16, 64, 128 and 256 rows from one build: 512^2 0.78, 0.80, 0.86; 2048^2 0.90, 0.92, 0.97; 4096^2
// 1.30, 1.20, 1.21; 8192^2 1.68, 1.64, 1.54).  Gram pairs and the products with them are 64-bit MFMAs whose operands are the registers
// the rows are in: S = sum over rows of (c u)(c u)^T with lane (rank, row) as both operands.
#pragma once

constexpr int kRunThreads = 1024, kRunWaves = kRunThreads / 64;
constexpr int kRunRows = 64, kRunScaleRows = 128, kRunMaxBlocks = kMaxShares;
constexpr int kSlot = 32;            // doubles per parity: beta [16], rho, pending factor of Y
constexpr uint32_t kStop = 0x80000000u;

struct PtqRun {
    double* partU[2];   // shares of the blocks of a Tikhonov step, [nbU, count]
    double* partS[2];   // the same of a scale step, [nbS, count]
    double* gf;         // [parity][side][nbU of the side, up to kRunMaxBlocks][2]: consensus gap and sign changes of a block
    double* slot;       // [parity][kSlot]
    uint32_t* sync;     // [kSyncWords], zero between launches
    int nbU[2], nbS[2], passU[2], passS[2];
    int t_begin, t_end;
};

struct PtqRunArgs {
    PtqArgs a;
    PtqRun g;
};

struct RunBlocks { int nb, pass; };
inline RunBlocks run_blocks(int64_t n, int rows) {
    RunBlocks b;
    b.pass = static_cast<int>((n + static_cast<int64_t>(rows) * kRunMaxBlocks - 1) / (static_cast<int64_t>(rows) * kRunMaxBlocks));
    b.nb = static_cast<int>((n + static_cast<int64_t>(rows) * b.pass - 1) / (static_cast<int64_t>(rows) * b.pass));
    return b;
}
// Values of a share: the lower triangle of S by rows, then K by rows.
__host__ __device__ constexpr int run_count(int R, int r0) { return R * (R + 1) / 2 + R * r0; }
// LDS of the run kernel in doubles: the two totals, the operands, beta and its work area, scales, the waves' shares.
constexpr int run_lds_doubles(int RT) {
    return 2 * (RT == 1 ? 512 : 768) + 256 + 256 * RT + 16 + (2 * 16 * 17 + 3 * 16 + 8) + 16 * (16 * RT + 1) + kRunWaves * 16 + 2 * kRunWaves + 8 + kRunWaves * 256 * (1 + RT);
}

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

// acc[e] += (lane K + e's `from`) * f[e], e = 0..3
template <int K>
__device__ inline void fma_row_lanes4(double (&acc)[4], double from, const double (&f)[4]) {
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %4, %5 row_newbcast:%c9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, %6 row_newbcast:%c10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, %7 row_newbcast:%c11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %4, %8 row_newbcast:%c12 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
        : "v"(from), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3));
}

// sum over c < 16 of M[c][l] * (lane c's f), M in LDS as pairs of rows
template <int C = 0>
__device__ inline void row_products(const double* M, double f, int l, double (&acc)[4]) {
    const d2 a = *reinterpret_cast<const d2*>(M + (C >> 1) * 32 + l * 2), b = *reinterpret_cast<const d2*>(M + ((C >> 1) + 1) * 32 + l * 2);
    const double m[4] = {a[0], a[1], b[0], b[1]};
    fma_row_lanes4<C>(acc, f, m);
    if constexpr (C < 12) row_products<C + 4>(M, f, l, acc);
}

// p[i] by a 32-bit byte offset from a uniform pointer: one address register per lane
template <class T>
__device__ inline T* at32(T* p, uint32_t i) {
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type Byte;
    return reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + i * static_cast<uint32_t>(sizeof(T)));
}

template <int RT>   // factor rank at most 16 RT
__global__ __launch_bounds__(kRunThreads) void lordba_ptq_run_kernel(PtqRunArgs) {
    constexpr int NT = 1 + RT;              // 16 x 16 tiles of a Gram pair
    constexpr int NV = RT == 1 ? 512 : 768; // threads that have a value each: at least run_count(16, 16 RT)
    constexpr int H = NV <= 512 ? 2 : 1;    // threads that share the sum of one value
    typedef const __attribute__((address_space(4))) PtqRunArgs KernelArgs;   // (constant memory: read into scalar registers)
    KernelArgs* arg = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const int R = arg->a.R, r0 = arg->a.r0, RP = R * (R + 1) / 2, count = run_count(R, r0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* T1 = lds;                  // totals of side 0 and of side 1, as they are stored (for beta)
    double* T2 = T1 + NV;
    double* G = T2 + NV;               // S as pairs of rows: entry (i, j) at (i / 2) * 32 + 2 j + i % 2, zeros beyond R
    double* Kt = G + 256;              // K transposed [16 RT, 16], the same way
    double* bs = Kt + 256 * RT;        // beta
    double* bw = bs + 16;              // beta_pinv_solve's areas
    double* hp = bw + 2 * 16 * 17 + 3 * 16 + 8;   // [16][16 RT + 1]: K1 o K2
    double* cs = hp + 16 * (16 * RT + 1);         // [waves][16]
    double* gfs = cs + kRunWaves * 16;            // [waves][2]
    double* ctl = gfs + 2 * kRunWaves;            // rho, factor of Y, done
    double* red = ctl + 8;                        // [waves][NV]
    __shared__ uint32_t sh_number[2], sh_numbers, sh_stop[2], place[NV];
    __shared__ uint32_t sh_over;
    int waits = 0;   // (two flags in turn: the next wait's must not be set before every wave has read this one's)

    // Value o of a Gram pair as it is stored: whether there is one (bit 0) and it belongs to S (1), its row and column (2..5, 6..10), its
    // place in G and Kt (11..20; S again at the mirrored place) and in a wave's share (21..30).
    for (int o = threadIdx.x; o < NV; o += kRunThreads) {
        const bool is_s = o < RP;
        int i = 0, j = o;
        if (is_s) {
            while (j > i) j -= ++i;
        } else {
            i = (o - RP) / r0;
            j = (o - RP) - i * r0;
        }
        const int at = is_s ? (i >> 1) * 32 + j * 2 + (i & 1) : 256 + (j >> 1) * 32 + i * 2 + (j & 1);
        const int rpos = is_s ? i * 16 + j : (1 + (j >> 4)) * 256 + i * 16 + (j & 15);
        place[o] = o < count ? 1u | (is_s ? 2u : 0u) | i << 2 | j << 6 | at << 11 | static_cast<uint32_t>(rpos) << 21 : 0u;
    }
    for (int o = threadIdx.x; o < 256 * NT; o += kRunThreads) G[o] = 0.0;   // (Kt follows G)
    if (threadIdx.x < 16) bs[threadIdx.x] = 0.0;
    auto arrivals = [&](int p) { return arg->g.sync + (2 + p) * kSyncStride; };
    uint32_t* const kept = arg->g.sync + kSyncKeeper;   // sweeps whose beta and penalty the keeper has published
    const bool init = arg->g.t_begin == 0;
    auto per = [&](int p) { return p == 0 ? arg->g.nbU[0] + 1 : p == 1 ? arg->g.nbU[1] : arg->g.nbS[p & 1]; };   // (the first step has a keeper: beta and the penalty)
    const uint32_t per_sweep = static_cast<uint32_t>(per(0) + per(1) + per(2) + per(3));
    const uint32_t n_init = init ? per_sweep - 1u : 0u;
    // How many numbers there are.  An update that has no carriers (or a run whose signs have repeated) makes no sweeps; the iterates are
    // still set.  Behind the last sweep comes one more number: beta and the penalty of that sweep.  One thread reads the end flag for the
    // workgroup: the keeper of this launch sets it too, and a workgroup that starts as the run ends must leave whole or stay whole (it may
    // see either value: everything before its number is done by then, and what it would wait for carries the stop bit or soon will).
    if (threadIdx.x == 0) {
        const uint32_t sweeps = static_cast<uint32_t>(arg->g.t_end - arg->g.t_begin);
        if (published(arg->a.ctrl + kDone) != 0.0) sh_numbers = init ? n_init - static_cast<uint32_t>(per(2) + per(3)) : 0u;
        else sh_numbers = n_init + (sweeps == 0u ? 0u : sweeps * per_sweep + 1u);
        sh_over = 0u;
        sh_number[0] = __hip_atomic_fetch_add(arg->g.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    auto need = [&](int p, int t) {   // arrivals of step p through sweep t
        const int base = !init ? 0 : p == 0 ? per(0) - 1 : per(p);
        return static_cast<uint32_t>(base + (t - arg->g.t_begin + 1) * per(p));
    };
    // Lane-derived values and arguments are taken anew in every block, from numbers that the compiler cannot follow: kept over the whole
    // kernel, with the lane masks of every phase that follow from them, they take more registers than there are, scalar ones above all.
    // (What is left: 36 vector registers in scratch memory, 84 bytes per lane, at factor ranks up to 16, 92 and 176 bytes beyond, and
    // 130 to 140 scalar ones in lanes of vector registers.)
    int tid = threadIdx.x;
    int turn = 0;
    uint32_t next = 0u;   // the first thread's next number: asked for while it works on the one before
    // The next number, asked for once the step before the present block's is seen to be complete: workgroups that end a step together queue
    // for it, 64 of them for 7 us.  Not before: what a workgroup holds while it still waits, nobody else can do meanwhile.  (Whoever holds a
    // number behind the one it works on does that one first, so the smallest unfinished number is still always being worked on.)
    auto ask = [&]() {
        if (tid == 0) next = __hip_atomic_fetch_add(arg->g.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto wait_for = [&](int p, int t) {   // true: the run is over
        uint32_t* stop = &sh_stop[waits++ & 1];
        if (tid == 0) {
            const uint32_t want = need(p, t);
            uint32_t v;
            while ((v = __hip_atomic_load(arrivals(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < want) __builtin_amdgcn_s_sleep(1);
            *stop = v & kStop;   // (with the stop bit the count is beyond any other)
        }
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(*stop) != 0u;
    };
    auto arrive = [&](int p, bool keeper = false) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        ++turn;
        if (tid == 0) sh_number[turn & 1] = next;   // (the other one may not have been read by every wave yet)
        __syncthreads();
        if (tid == 0) {
            __hip_atomic_fetch_add(arrivals(p), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (keeper) __hip_atomic_fetch_add(kept, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // This thread's share of the sum over the blocks.  With mark < 2 the shares may still be on their way and are taken as they come, by
    // the sweep's mark that they carry: first one of them alone, until it is there (or the run is over: sh_over), then all.  want_kept:
    // how many sweeps' beta must have been published too.
    auto gather = [&](const double* part, int nb, uint32_t mark, int blk, uint32_t want_kept) {
        const int o = H == 2 ? tid & (NV - 1) : tid, h = H == 2 ? wave / (NV / 64) : 0;
        const int lo = h == 1 ? (nb + 1) >> 1 : 0, hi = H == 2 && h == 0 ? (nb + 1) >> 1 : nb;   // (the first wave always has a block)
        if ((H == 2 ? (wave * 64) & (NV - 1) : wave * 64) >= count || lo == hi) return 0.0;   // (scalar)
        const uint32_t oc = static_cast<uint32_t>(o < count ? o : count - 1);
        if (mark < 2u) {
            const double* one = part + (lo + blk % (hi - lo)) * count;
            for (;;) {   // (one wave alone reads the keeper's word for the workgroup: all of them together crowd its memory channel)
                uint32_t k = want_kept;
                if (wave == 0) k = __hip_atomic_load(kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool other = other_mark(mark_word(published(at32(one, oc)), mark));
                if (wave == 0 && (k & kStop)) { sh_over = 1u; return 0.0; }
                if (__builtin_amdgcn_ballot_w64(other || k < want_kept) == 0ull) break;
                if (__hip_atomic_load(&sh_over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u) return 0.0;
                __builtin_amdgcn_s_sleep(1);
            }
        }
        double acc = 0.0;
        for (int b0 = lo; b0 < hi; b0 += 16) {
            double v[16];
            uint32_t word;
            do {   // (shares of one step arrive close together: this seldom takes more than two turns)
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] = published(at32(part + (b0 + j < hi ? b0 + j : hi - 1) * count, oc));
                word = 0u;
#pragma unroll
                for (int j = 0; j < 16; ++j) word |= mark_word(v[j], mark);
            } while (mark < 2u && __builtin_amdgcn_ballot_w64(other_mark(word)) != 0ull);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc = fma(b0 + j < hi ? without_mark(v[j]) : 0.0, kShareUnit, acc);
        }
        return o < count ? share_sum(acc) : 0.0;
    };
    auto combine = [&](double acc) {   // the whole sum, in the threads below NV (contains a barrier)
        if constexpr (H == 2) {
            if (tid >= NV) red[tid - NV] = acc;
            __syncthreads();
            if (tid < NV) acc += red[tid];
        }
        return acc;
    };
    // the waves' shares added up and published with the sweep's mark (contains a barrier)
    auto share = [&](const d4 (&s)[NT], double* part, uint32_t mark) {
#pragma unroll
        for (int e = 0; e < NT; ++e) {
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * NT + e) * 256 + r * 64 + (tid & 63)] = s[e][r];
        }
        __syncthreads();
        if (tid < count) {
            const double* at = red + (place[tid] >> 21);
            double v[kRunWaves], acc = 0.0;
#pragma unroll
            for (int w = 0; w < kRunWaves; ++w) v[w] = at[w * NT * 256];
#pragma unroll
            for (int w = 0; w < kRunWaves; ++w) acc += v[w];
            publish(part + tid, with_mark(acc, mark));
        }
    };

    for (;;) {
        asm volatile("" : "+v"(tid));
        asm volatile("" : "+s"(arg));
        const int lane = tid & 63, li = lane & 15, q = lane >> 4;
        uint32_t rest = __builtin_amdgcn_readfirstlane(sh_number[turn & 1]);
        if (rest >= __builtin_amdgcn_readfirstlane(sh_numbers)) break;
        int t = -1, p = 0;
        if (rest >= n_init) {
            rest -= n_init;
            const uint32_t s = rest / per_sweep;
            rest -= s * per_sweep;
            t = arg->g.t_begin + static_cast<int>(s);
        } else {
            ++rest;   // (the warm start has no keeper)
        }
        for (; rest >= static_cast<uint32_t>(per(p)); ++p) rest -= static_cast<uint32_t>(per(p));
        // The keeper comes first: the blocks behind it may leave when they see that the run is over, it tells the others.
        const bool keeper = p == 0 && rest == 0u;
        const int blk = static_cast<int>(rest) - (p == 0 && !keeper ? 1 : 0), side = p & 1;
        const int64_t n = arg->a.n[side];
        const __half* F = arg->a.F[side];
        auto factor = [&](int64_t row, int c) {   // entry c of a factor row; zeros beyond the rows and the rank
            const bool in = row < n && c < r0;
            const float v = __half2float(F[in ? row * r0 + c : 0]);
            return in ? static_cast<double>(v) : 0.0;
        };

        if (p < 2 && t < 0) {   // ---- warm start: U = M = sign(factor row . Z), Y = 0, scale = 1
            d4 s[NT];
#pragma unroll
            for (int e = 0; e < NT; ++e) s[e] = d4{0.0, 0.0, 0.0, 0.0};
            for (int pass = 0; pass < arg->g.passU[side]; ++pass) {
                const int64_t row = (static_cast<int64_t>(blk) * arg->g.passU[side] + pass) * kRunRows + wave * 4 + q;
                const bool in = row < n, act = in && li < R;
                double acc = 0.0;
                for (int c = 0; c < r0; ++c) acc += factor(row, c) * arg->a.Z[side][c * R + (li < R ? li : 0)];
                const double v = act ? (acc < 0.0 ? -1.0 : 1.0) : 0.0;
                if (act) {
                    publish(arg->a.X[side] + row * R + li, v);
                    publish(arg->a.Mm[side] + row * R + li, v);
                    publish(arg->a.Y[side] + row * R + li, 0.0);
                }
                if (in && li == 0) publish(arg->a.scale[side] + row, 1.0);
                s[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, s[0], 0, 0, 0);
#pragma unroll
                for (int e = 0; e < RT; ++e) s[1 + e] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, factor(row, e * 16 + li), s[1 + e], 0, 0, 0);
            }
            ask();
            if (side == 1) share(s, arg->g.partU[1] + static_cast<int64_t>(blk) * count, t & 1);   // (all that alpha needs)
            arrive(p);
            continue;
        }
        if (p < 2) {   // ---- Tikhonov step of a side, signs and duals; before U1's, beta and the penalty of the sweep before
            const bool update = p == 0 && t > arg->g.t_begin;
            const bool marked = t > arg->g.t_begin + (p == 0 ? 1 : 0);   // (the shares it waits for are not the first in their place)
            double acc1 = 0.0;
            if (update) {
                // U2's step of the sweep before: its consensus gaps, which are published behind its shares.  (The shares of alpha's step that lie in
                // their place are then those of one sweep earlier, whose mark is the other one, not of two.)
                if (wait_for(1, t - 1)) break;
                if (marked) {
                    acc1 = combine(gather(arg->g.partS[0], arg->g.nbS[0], static_cast<uint32_t>(t - 1) & 1u, blk, 0u));
                    if (H == 1) __syncthreads();
                    if (__builtin_amdgcn_readfirstlane(sh_over) != 0u) break;
                }
            }
            if (wait_for(p + 2, t - 1)) break;
            // what the rows need is there already: requested ahead of the wait for the totals
            const int passes = keeper ? 0 : arg->g.passU[side];
            double m_old = 0.0, y_old = 0.0, c = 0.0, f[RT];
            auto request = [&](int pass) {
                const int64_t row = (static_cast<int64_t>(blk) * passes + pass) * kRunRows + wave * 4 + q;
                const bool in = row < n && passes > 0;
                const int64_t at = in ? row * R + (li < R ? li : 0) : 0;
                m_old = published(arg->a.Mm[side] + at);
                y_old = published(arg->a.Y[side] + at);
                c = published(arg->a.scale[side] + (in ? row : 0));
#pragma unroll
                for (int e = 0; e < RT; ++e) f[e] = factor(in ? row : n, e * 16 + li);
                c = in ? c : 0.0;
            };
            request(0);
            if (update) {
                if (!marked) acc1 = combine(gather(arg->g.partS[0], arg->g.nbS[0], 2u, 0, 0u));
                if (tid < count) T1[tid] = acc1;
                if (wave == 1) {   // consensus gaps and sign changes of both sides
                    double gap = 0.0, f0 = 0.0, f1 = 0.0;
                    const double* gf = arg->g.gf + ((t - 1) & 1) * 4 * kRunMaxBlocks;
                    if (lane < arg->g.nbU[0]) { gap += published(gf + 2 * lane); f0 = published(gf + 2 * lane + 1); }
                    gf += 2 * kRunMaxBlocks;
                    if (lane < arg->g.nbU[1]) { gap += published(gf + 2 * lane); f1 = published(gf + 2 * lane + 1); }
                    gap = group_sum(gap, 64);
                    f0 = group_sum(f0, 64);
                    f1 = group_sum(f1, 64);
                    if (lane == 0) {
                        const double* slot = arg->g.slot + ((t - 1) & 1) * kSlot;
                        double rho = published(slot + 16), yfac = 1.0;
                        if (2 * static_cast<int64_t>(t - 1) < arg->a.K) {   // residual balancing in the first half of the run
                            const double rho0 = rho / (static_cast<double>(arg->a.n[0]) * R), rho1 = rho / (static_cast<double>(arg->a.n[1]) * R);
                            const double rp = sqrt(gap), sd = sqrt(rho0 * rho0 * 4.0 * f0 + rho1 * rho1 * 4.0 * f1);
                            if (rp > arg->a.mu * sd) { rho *= arg->a.tau; yfac = 1.0 / arg->a.tau; }
                            else if (sd > arg->a.mu * rp) { rho /= arg->a.tau; yfac = arg->a.tau; }
                        }
                        ctl[0] = rho;
                        ctl[1] = yfac;
                        ctl[2] = f0 + f1 == 0.0 ? 1.0 : 0.0;
                    }
                }
            }
            if (!marked) {
                if (p == 0 ? wait_for(3, t - 1) : wait_for(0, t)) break;
            }
            double total = gather(p == 0 ? arg->g.partS[1] : arg->g.partU[0], p == 0 ? arg->g.nbS[1] : arg->g.nbU[0],
                                  marked ? static_cast<uint32_t>(p == 0 ? t - 1 : t) & 1u : 2u, blk, p == 0 ? 0u : static_cast<uint32_t>(t - arg->g.t_begin + 1));
            if (!update && tid < 18) {   // beta, rho, factor of Y
                double v;
                if (p == 0) v = tid < 16 ? (tid < R ? arg->a.beta[tid] : 0.0) : arg->a.ctrl[tid == 16 ? kRho : kYfac];
                else v = published(arg->g.slot + (t & 1) * kSlot + tid);
                if (tid < 16) bs[tid] = v;
                else ctl[tid - 16] = v;
            }
            ask();
            total = combine(total);
            if (H == 1) __syncthreads();
            if (marked && __builtin_amdgcn_readfirstlane(sh_over) != 0u) break;
            if (update) {
                double* Gb = bw;
                double* N2 = Gb + 16 * 17;
                double* hv = N2 + 16 * 17;
                double* bt = hv + 16;
                int* perm = reinterpret_cast<int*>(bt + 16);
                const int ld = R + 1;
                // Eq. (beta-gram), Eq. (beta-pinv): beta = pinv(S1 o S2) h, h_k = K1[k, :] . K2[k, :]
                if (tid < count) {
                    const uint32_t w = place[tid];
                    const int i = w >> 2 & 15u, j = w >> 6 & 31u;
                    T2[tid] = total;
                    *(w & 2u ? Gb + i * ld + j : hp + i * (16 * RT + 1) + j) = acc1 * total;
                    if (w & 2u) Gb[j * ld + i] = acc1 * total;
                }
                __syncthreads();
                if (wave == 0) {
                    const int k = lane >> 2;   // four lanes per entry of h
                    double h = 0.0;
#pragma unroll
                    for (int c = 0; c < 4 * RT; ++c) {
                        const int at = (lane & 3) + 4 * c;
                        const double v = hp[k * (16 * RT + 1) + at];
                        h += at < r0 ? v : 0.0;
                    }
                    h += dpp_move<0xb1>(h);   // (among the four lanes)
                    h += dpp_move<0x4e>(h);
                    if (k < R && (lane & 3) == 0) hv[k] = h;
                    if (lane < R) perm[lane] = lane;
                    wave_sync();
                    beta_pinv_solve(Gb, ld, hv, N2, perm, bt, R, lane);
                    if (lane < R) bs[lane] = bt[lane];
                }
                __syncthreads();
            }
            if (tid < count) {
                const uint32_t w = place[tid];
                const int i = w >> 2 & 15u, j = w >> 6 & 31u;
                const double v = total * (bs[i] * (w & 2u ? bs[j] : 1.0));
                G[w >> 11 & 0x3ffu] = v;
                if (w & 2u) G[(j >> 1) * 32 + i * 2 + (j & 1)] = v;
            }
            if (keeper) {
                const bool done = update && ctl[2] != 0.0, last = done || t == arg->g.t_end;
                if (tid < 18) publish(arg->g.slot + (t & 1) * kSlot + tid, tid < 16 ? bs[tid] : ctl[tid - 16]);
                if (update && wave == 0) {   // objective of Eq. (admm-problem): (||T||_F^2 - 2 beta . h + beta^T G beta) / 2
                    double lin = 0.0, quad = 0.0;
                    if (lane < R) {
                        const double bl = bs[lane];
                        for (int e = 0; e < r0; ++e) lin += T1[RP + lane * r0 + e] * T2[RP + lane * r0 + e];
                        lin *= bl;
                        for (int i = 0; i < R; ++i) {
                            const int hi = i > lane ? i : lane, at = hi * (hi + 1) / 2 + (i > lane ? lane : i);
                            quad += bl * bs[i] * (T1[at] * T2[at]);
                        }
                    }
                    lin = group_sum(lin, 64);
                    quad = group_sum(quad, 64);
                    if (lane == 0) arg->a.info[kInfoHead + t - 1] = 0.5 * (arg->a.ctrl[kNormT2] - 2.0 * lin + quad);
                    if (last) {
                        if (lane < R) arg->a.beta[lane] = bs[lane];
                        if (lane == 0) {
                            arg->a.ctrl[kRho] = ctl[0];
                            arg->a.ctrl[kYfac] = ctl[1];
                            arg->a.ctrl[kSweeps] = t;
                            if (done) { arg->a.ctrl[kFrozen] = 1.0; arg->a.ctrl[kDone] = 1.0; }
                        }
                    }
                }
                if (last) {   // nobody arrives at this step any more; where the run is over, the others may be waiting
                    if (done && tid < 5) __hip_atomic_fetch_or(tid < 4 ? arrivals(tid) : kept, kStop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (before this workgroup counts as gone: whoever leaves last sets the bits back)
                    break;
                }
                arrive(0, true);
                continue;
            }
            if (update && ctl[2] != 0.0) break;
            __syncthreads();
            const double rho_k = ctl[0] / (static_cast<double>(n) * R), yfac = ctl[1];
            d4 s[NT];
#pragma unroll
            for (int e = 0; e < NT; ++e) s[e] = d4{0.0, 0.0, 0.0, 0.0};
            double gap = 0.0, flips = 0.0;
            const bool act = li < R;
            for (int pass = 0; pass < passes; ++pass) {
                const int64_t row = (static_cast<int64_t>(blk) * passes + pass) * kRunRows + wave * 4 + q;
                const bool in = row < n;
                double kb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < RT; ++e) row_products(Kt + e * 256, f[e], li, kb);
                const double y = yfac * y_old, mo = m_old, cc = c;
                double b = act ? cc * ((kb[0] + kb[1]) + (kb[2] + kb[3])) + rho_k * (mo - y) : 0.0;
                const double c2 = cc * cc;
                double col[16];
                const double* Gl = G + li * 2;
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const d2 gg = *reinterpret_cast<const d2*>(Gl + i * 16);
                    col[i] = c2 * gg[0];
                    col[i + 1] = c2 * gg[1];
                }
                double fr[RT];
#pragma unroll
                for (int e = 0; e < RT; ++e) fr[e] = f[e];
                if (pass + 1 < passes) request(pass + 1);
                double pivot;   // positive: the matrix is a Gram matrix plus rho_k I
                const double x = row_ldlt_solve(col, b, rho_k, li, &pivot);
                const double mn = (x + y) < 0.0 ? -1.0 : 1.0;
                const bool live = in && act;
                if (live) {
                    publish(arg->a.X[side] + row * R + li, x);
                    publish(arg->a.Mm[side] + row * R + li, mn);
                    publish(arg->a.Y[side] + row * R + li, y + x - mn);
                    gap += (x - mn) * (x - mn);
                    flips += mn != mo ? 1.0 : 0.0;
                }
                const double v = live ? cc * x : 0.0;
                s[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, s[0], 0, 0, 0);
#pragma unroll
                for (int e = 0; e < RT; ++e) s[1 + e] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, fr[e], s[1 + e], 0, 0, 0);
            }
            share(s, arg->g.partU[side] + static_cast<int64_t>(blk) * count, t & 1);
            gap = group_sum(gap, 64);
            flips = group_sum(flips, 64);
            if (lane == 0) { gfs[2 * wave] = gap; gfs[2 * wave + 1] = flips; }
            __syncthreads();
            if (tid >= kRunThreads - 64 && lane < 2) {   // (a wave without a value to add up where there are 512)
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < kRunWaves; ++w) sum += gfs[2 * w + lane];
                publish(arg->g.gf + (((t & 1) * 2 + side) * kRunMaxBlocks + blk) * 2 + lane, sum);
            }
            arrive(p);
            continue;
        }
        // ---- Eq. (alpha-update), Eq. (gamma-update): per row, with v = u o beta, (v . (K f)) / (v^T S v), 0 where the denominator is 0
        if (p == 2 ? wait_for(0, t) : wait_for(1, t)) break;
        const int passes = arg->g.passS[side];
        double xr[4], xk[4];   // the wave's 16 rows by lane (row, ranks 4 s + q) and by lane (rank, rows 4 s + q)
        __half fr[RT][4], fk[RT][4];
        auto request = [&](int pass) {   // (what is not there is read from the first row and dropped where it is used)
            const int64_t row0 = (static_cast<int64_t>(blk) * passes + pass) * kRunScaleRows + wave * 16;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int64_t r1 = row0 + li, r2 = row0 + 4 * s + q;
                const int k = 4 * s + q;
                xr[s] = published(arg->a.X[side] + (r1 < n && k < R ? r1 * R + k : 0));
                xk[s] = published(arg->a.X[side] + (r2 < n && li < R ? r2 * R + li : 0));
#pragma unroll
                for (int e = 0; e < RT; ++e) {
                    fr[e][s] = F[r1 < n && e * 16 + k < r0 ? r1 * r0 + e * 16 + k : 0];
                    fk[e][s] = F[r2 < n && e * 16 + li < r0 ? r2 * r0 + e * 16 + li : 0];
                }
            }
        };
        const bool rows_here = wave < kRunScaleRows / 16;   // (the other waves only add shares up)
        double beta_k = 0.0;
        if (tid < 16) beta_k = t < 0 ? (tid < R ? arg->a.beta[tid] : 0.0) : published(arg->g.slot + (t & 1) * kSlot + tid);
        if (rows_here) request(0);
        if (tid < 16) bs[tid] = beta_k;
        const bool marked = t > arg->g.t_begin;
        if (!marked && wait_for(p - 1, t)) break;
        {
            const double mine = gather(p == 2 ? arg->g.partU[1] : arg->g.partS[0], p == 2 ? arg->g.nbU[1] : arg->g.nbS[0], marked ? t & 1 : 2u, blk, 0u);
            ask();
            const double total = combine(mine);
            if (tid < count) {
                const uint32_t w = place[tid];
                const int i = w >> 2 & 15u, j = w >> 6 & 31u;
                G[w >> 11 & 0x3ffu] = total;
                if (w & 2u) G[(j >> 1) * 32 + i * 2 + (j & 1)] = total;
            }
        }
        __syncthreads();
        if (marked && __builtin_amdgcn_readfirstlane(sh_over) != 0u) break;
        d4 s[NT];
#pragma unroll
        for (int e = 0; e < NT; ++e) s[e] = d4{0.0, 0.0, 0.0, 0.0};
        for (int pass = 0; pass < passes && rows_here; ++pass) {
            const int64_t row = (static_cast<int64_t>(blk) * passes + pass) * kRunScaleRows + wave * 16 + li;
            const bool in = row < n;
            d4 sv = {0.0, 0.0, 0.0, 0.0}, kf = {0.0, 0.0, 0.0, 0.0};
            double v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // ranks 4 e + q: operand (rank, q) of S, which is symmetric, and of K
                const int k = 4 * e + q;
                v[e] = in && k < R ? xr[e] * bs[k] : 0.0;
                sv = __builtin_amdgcn_mfma_f64_16x16x4f64(G[(k >> 1) * 32 + li * 2 + (k & 1)], v[e], sv, 0, 0, 0);
#pragma unroll
                for (int w = 0; w < RT; ++w)
                    kf = __builtin_amdgcn_mfma_f64_16x16x4f64(Kt[w * 256 + (k >> 1) * 32 + li * 2 + (k & 1)],
                                                              in && w * 16 + k < r0 ? static_cast<double>(__half2float(fr[w][e])) : 0.0, kf, 0, 0, 0);
            }
            double num = 0.0, den = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                num = fma(v[e], kf[e], num);
                den = fma(v[e], sv[e], den);
            }
            num += __shfl_xor(num, 16, 64);
            den += __shfl_xor(den, 16, 64);
            num += __shfl_xor(num, 32, 64);
            den += __shfl_xor(den, 32, 64);
            const double c = den > 0.0 ? num / den : 0.0;
            wave_sync();
            if (q == 0) {
                cs[wave * 16 + li] = in ? c : 0.0;
                if (in) publish(arg->a.scale[side] + row, c);
            }
            wave_sync();
            double u[4], fv[RT][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool ink = row - li + 4 * e + q < n;
                u[e] = ink && li < R ? cs[wave * 16 + 4 * e + q] * xk[e] : 0.0;
#pragma unroll
                for (int w = 0; w < RT; ++w) fv[w][e] = ink && w * 16 + li < r0 ? static_cast<double>(__half2float(fk[w][e])) : 0.0;
            }
            if (pass + 1 < passes) request(pass + 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[e], u[e], s[0], 0, 0, 0);
#pragma unroll
                for (int w = 0; w < RT; ++w) s[1 + w] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[e], fv[w][e], s[1 + w], 0, 0, 0);
            }
        }
        share(s, arg->g.partS[side] + static_cast<int64_t>(blk) * count, t & 1);
        arrive(p);
    }
    // The last workgroup to leave sets the counters back for the next launch: by then nobody reads them, and nothing written to them (the
    // numbers asked for ahead too) is still under way.
    if (tid == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (__hip_atomic_fetch_add(arg->g.sync + kSyncStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x) {
            for (int e = 0; e < 6; ++e) __hip_atomic_store(arg->g.sync + e * kSyncStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(kept, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}
