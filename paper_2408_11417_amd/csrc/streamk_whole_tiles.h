// The four-wave kernel for plans without split tiles, 16-byte aligned rows and 16-bit output: the MAC loop runs on from
// one tile of a workgroup to the next.
//
// What bounds such plans besides the MAC loop is what lies between two tiles of a workgroup: in streamk_gemm_kernel
// the ring of LDS stages drains, the tile is converted and stored while the matrix cores idle (all workgroups at the
// same moment: 256 tiles of 256 x 256 are 32 MB, 6 us at the rate HBM takes writes), and the ring fills again.  Here
//  - the requests of a tile's last k-iterations are those of the next tile's first ones, so the ring never drains;
//  - the finished blocks are packed to 16 bits among the last matrix-core instructions of their tile and the
//    accumulators start from zero with the next one's first k-step;
//  - the packed blocks stay in registers (128 per lane with 16-bit operands) and leave in the following trips, one pair of
//    blocks per trip, their lane exchange and their stores in the shadow of the matrix-core work.
// With operands in turn, against what ran before it, us: 8192 x 8192 x 512 bf16 82.0 -> 77.8 (N(0, 1/K) values; uniform ones 79 - 81 -> 76 - 80
// on five boxes, one of which showed no gain), 12288 x 12288 x 1024 283.5 -> 269.2, 8192^3 750 -> 737; 8 bits 8192 x 8192 x 1024
// 103.2 -> 73.7, 8192^3 374 -> 357.  One tile per workgroup gains from the trips alone (one offset per operand and lane, 5
// instructions per request): 3840 x 4224 x 4096 bf16 104.8 -> 102.8, 8 bits 4096 x 4096 x 640 26.5 -> 18.2 (tile forced).
// Counters, before -> now: 8192 x 8192 x 512 172 -> 156 thousand cycles at 2.08 -> 2.16 GHz, matrix cores busy 0.38 -> 0.42 (they need 65.5:
// the rest is not the clock); 8192^3 1.306 -> 1.265 million at 1.61 -> 1.58 GHz, busy 0.80 -> 0.83; 8 bits 0.719 -> 0.644
// at 1.78 -> 1.67, 0.73 -> 0.81.
// A long K is bound by the power limit: most of the cycles saved come back as a lower clock.
//
// The accumulators fill the 256 accumulation registers, so the code is laid out for a register allocation in place: one
// loop nest that makes and ends them once per tile (a second copy of a tile's end, or packing beside the next tile's
// first instructions, spilled 600 registers).  The 16-bit kernels spill 3 vector registers (12 bytes of scratch per lane) and 94 scalar ones,
// the 8-bit kernel 54 scalar ones.  The steady trip holds none of them, but the trip that hands over a ragged k-iteration reloads one
// from scratch and so waits for all requests, once per tile whose K is not a multiple of BK.
#pragma once
#include "streamk_kernels.h"

namespace streamk_detail {


template <class C> struct WholeTiles {
    static_assert(C::FINE && C::NSA == C::NSB + 1 && C::MF == 32 && C::NI % 2 == 0 && C::KK % 2 == 0 && C::A_WAVES == C::NW, "layout of the kernel");
    static constexpr int NM = C::MI * C::NI, SLOTS = C::KK * NM;       // matrix-core instructions of a k-step, of a trip
    static constexpr int PAIRS = NM / 2;                               // pairs of blocks = trips that store
    static constexpr int PAIR_STORES = 4;
    // pairs kept in registers (16 each) beside the two operand sets and some 60 others: all eight with 16-bit operands, four in 8
    // bits.  The others leave at once.
    static constexpr int KEPT = (256 - 60 - 2 * C::FRAG_REGS) / 16 < PAIRS ? (256 - 60 - 2 * C::FRAG_REGS) / 16 : PAIRS;
    static constexpr int TAKEN_LATE = 4;                               // a block is packed that many matrix-core instructions after its last one
    // pairs that leave at once behind the last request of B of the trip (which is among the first k-step's if there are two)
    static constexpr int after_requests() {
        int n = 0;
        for (int p = KEPT; p < PAIRS; p++) n += 2 * p + 1 + TAKEN_LATE >= NM - 1;
        return n;
    }
    static_assert(KEPT == PAIRS || C::KK == 2, "all requests of B are out when the turn's k-step ends");
    static constexpr int CHECKED = C::NSA + 2;                         // a tile's last trips: requests cross into a ragged k-iteration and the next tile
    static constexpr int MIN_ITERS = KEPT < CHECKED ? CHECKED : KEPT;                        // the kept pairs leave in as many trips before the next turn
    static_assert((C::LPS * 8) % SLOTS == 0 || SLOTS % C::LPS == 0, "requests spread over the slots");
    static_assert(SLOTS % 16 == 0, "eight places for stores in the second half of a trip, of which the six phases take six");
};

template <class C, int OUT>
__device__ __forceinline__ void whole_tiles(const GemmArgs& g, unsigned char* smem) {
    typedef WholeTiles<C> W;
    typedef typename Mfma<C::DT, C::MF>::Acc Acc;
    constexpr int NM = W::NM, SLOTS = W::SLOTS, KK = C::KK;
    typedef std::true_type Yes;
    typedef std::false_type No;
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int x = logical_wg(blockIdx.x, g);
    const uint32_t lds0 = (uint32_t)(size_t)(lds_byte*)smem;
    const int nk = g.ipt, full_k = g.K / C::BK;        // k-iterations of a tile; those that lie wholly inside K
    FragMap<C> fm;
    fm.init();

    // this workgroup's tiles: the whole tiles of its Stream-K range and its data-parallel tiles
    int sk = x * g.ipw, sk_end = sk + g.ipw, dp_tile = g.sk_tiles + x;
    if (sk > g.sk_iters) sk = g.sk_iters;
    if (sk_end > g.sk_iters) sk_end = g.sk_iters;
    auto next_tile = [&](int& m0, int& n0) -> bool {
        const bool dp_now = dp_tile < g.tiles && (g.dp_first || sk >= sk_end);
        int tile;
        if (dp_now) {
            tile = dp_tile;
            dp_tile += g.grid;
        } else if (sk < sk_end) {
            tile = (int)fast_div((uint32_t)sk, g.div_ipt);
            sk += g.ipt;
        } else {
            return false;
        }
        int tm, tn;
        tile_position(g, tile, tm, tn);
        m0 = tm * C::BM;
        n0 = tn * C::BN;
        return true;
    };

    // ---- requests: one cursor for A and one, a stage behind, for B; they run on from tile to tile.  Request j of a wave
    // takes A_ROWS (B_ROWS) rows further down than request 0, at the same columns, so one offset per lane does for all
    // of a stage; beyond the last row of A, and the last row of B in a ragged k-iteration, it stays at that row.
    constexpr int A_ROWS = C::THREADS / C::CPA, B_ROWS = C::THREADS / C::CPB;
    static_assert(A_ROWS % 16 == 0 && B_ROWS % 8 == 0, "the swizzle of a lane's pieces is the same in every request");
    const char *a_base = static_cast<const char*>(g.A), *b_base = static_cast<const char*>(g.B);
    uint32_t a_off, a_max, b_off, b_max;               // byte offsets from a_base and b_base: of request 0, and where they stop
    int a_kit = 0, b_kit = 0;
    const int a_row = tid / C::CPA, a_col = C::PE * ((tid % C::CPA) ^ swz_a<C::CPA>(tid / C::CPA));
    const int b_row = tid / C::CPB, b_col = C::PE * ((tid % C::CPB) ^ swz_b<C::FP8, C::CPB>(tid / C::CPB));
    auto map_a = [&](int m0) {
        a_off = ((uint32_t)(m0 + a_row) * (uint32_t)g.K + (uint32_t)a_col) * C::ES;
        a_max = ((uint32_t)(g.M - 1) * (uint32_t)g.K + (uint32_t)a_col) * C::ES;
    };
    auto map_b = [&](int n0) {
        const int col = n0 + b_col < g.N ? n0 + b_col : g.N - C::PE;
        b_off = ((uint32_t)b_row * (uint32_t)g.N + (uint32_t)col) * C::ES;
        b_max = ~0u;
    };
    int m0, n0, m0_next = 0, n0_next = 0;
    if (!next_tile(m0, n0)) return;
    bool more = next_tile(m0_next, n0_next);
    // After the requests of a k-iteration: on to the next one.  In a last, ragged one pieces beyond K come from its first
    // columns (last row) instead and are cleared in LDS before they are used.  Beyond the last tile the requests go on (the
    // wait counts then hold to the end), all lanes for the same 16 bytes.  check: false in trips that are not among the last
    // CHECKED of a tile, in which none of this happens.
    auto advance_a = [&](bool check) {
        a_kit++;
        a_base += C::BK * C::ES;
        if (__builtin_expect(!check, 1)) return;
        if (a_kit == full_k && full_k < nk) {
            if (full_k * C::BK + a_col >= g.K) { a_off -= a_col * C::ES; a_max -= a_col * C::ES; }
        } else if (a_kit == nk) {
            a_base = static_cast<const char*>(g.A);
            a_kit = 0;
            if (more) map_a(m0_next);
            else a_max = 0;
        }
    };
    auto advance_b = [&](bool check) {
        b_kit++;
        b_base += (size_t)((uint32_t)(C::BK * C::ES)) * (uint32_t)g.N;
        if (__builtin_expect(!check, 1)) return;
        if (b_kit == full_k && full_k < nk) {
            b_max = b_off + (uint32_t)(g.K - 1 - full_k * C::BK - b_row) * (uint32_t)g.N * C::ES;
        } else if (b_kit == nk) {
            b_base = static_cast<const char*>(g.B);
            b_kit = 0;
            if (more) map_b(n0_next);
            else b_max = 0;
        }
    };
    const uint32_t a_step = (uint32_t)(A_ROWS * C::ES) * (uint32_t)g.K, b_step = (uint32_t)(B_ROWS * C::ES) * (uint32_t)g.N;
    auto request_a = [&](int j, int slot) {
        const uint32_t off = a_off + (uint32_t)j * a_step;
        lds_dma16(a_base, off < a_max ? off : a_max, lds0 + slot * C::A_BYTES + (j * C::NW + wave) * 1024);
    };
    auto request_b = [&](int j, int slot) {
        const uint32_t off = b_off + (uint32_t)j * b_step;
        lds_dma16(b_base, off < b_max ? off : b_max, lds0 + C::B_RING + slot * C::B_BYTES + (j * C::NW + wave) * 1024);
    };
    // requests q0 .. q1 - 1 of a trip: a stage of B, then one of A
    auto requests = [&](int q0, int q1, int slot_a, int slot_b) {
#pragma unroll
        for (int q = q0; q < q1; q++) {
            if (q < C::B_LD) request_b(q, slot_b);
            else request_a(q - C::B_LD, slot_a);
        }
    };

    // ---- results: the blocks of the previous tile, packed, and where they go (stores that lie beyond the end of the buffer
    // are dropped by the hardware: edge tiles need no branches)
    u32x4 out[W::KEPT][2][2];
    buffer_rsrc d_rsrc;
    uint32_t d_off[2];                                 // byte offset of this lane's first store of an even / odd pair of blocks
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int d_slot = lane / 32 + 2 * (lane / 16 % 2) + 4 * (lane / 8 % 2);
    auto pack_block = [&](const Acc& blk, u32x4 (&to)[2]) {
        auto pk = [](float lo, float hi) { return OUT == SK_BF16 ? pack_bf16(lo, hi) : pack_f16(lo, hi); };
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = 8 * h;
            const u32x2 d0 = __builtin_amdgcn_permlane32_swap(pk(blk[q], blk[q + 1]), pk(blk[q + 4], blk[q + 5]), false, false);
            const u32x2 d1 = __builtin_amdgcn_permlane32_swap(pk(blk[q + 2], blk[q + 3]), pk(blk[q + 6], blk[q + 7]), false, false);
            to[h] = u32x4{d0[0], d1[0], d0[1], d1[1]};
            asm volatile("" : "+v"(to[h]));            // (the accumulation registers are full)
        }
    };
    // the tile at m0, n0 is the one that leaves: its rows start at the descriptor's base, and what lies beyond row M - 1 is
    // beyond the descriptor's end; lanes beyond column N - 1 get an offset that always is
    auto aim = [&]() {
        const size_t first = (size_t)((uint32_t)m0 * (uint32_t)g.N + (uint32_t)n0);
        const int rows = g.M - m0 < C::BM ? g.M - m0 : C::BM;
        d_rsrc = __builtin_amdgcn_make_buffer_rsrc(static_cast<u16*>(g.D) + first, 0, (uint32_t)(rows * g.N - n0) * 2u, BUFFER_RAW);
#pragma unroll
        for (int p = 0; p < 2; p++) {
            const int col = wn * C::WTN + p * 64 + 8 * d_slot;
            d_off[p] = n0 + col < g.N ? ((uint32_t)(wm * C::WTM + lane % 8) * (uint32_t)g.N + (uint32_t)col) * 2u : 0x80000000u;
        }
    };
    // A pair of blocks side by side, in six phases: store_blocks' exchange, 8 rows of 128 bytes per store.
    u32x4 w00, w01, w10, w11, got;
    auto store_phase = [&](int pair, const u32x4 (&blks)[2][2], auto phase_number) {
        static_assert(C::NI == 4, "two pairs of blocks per block row");
        constexpr int phase = decltype(phase_number)::value;
        const bool upper8 = (lane & 8) != 0;
        auto exchange = [&](u32x4 x, u32x4 y, u32x4& lo, u32x4& hi) {
            const u32x2 d0 = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false), d1 = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
            const u32x2 d2 = __builtin_amdgcn_permlane16_swap(x[2], y[2], false, false), d3 = __builtin_amdgcn_permlane16_swap(x[3], y[3], false, false);
            lo = u32x4{d0[0], d1[0], d2[0], d3[0]};
            hi = u32x4{d0[1], d1[1], d2[1], d3[1]};
        };
        auto put = [&](u32x4 x, u32x4 y) {
            u32x4 v;
            if constexpr (phase % 2 == 0) {
                got = u32x4{swap_lane8(upper8 ? x[0] : y[0]), swap_lane8(upper8 ? x[1] : y[1]), swap_lane8(upper8 ? x[2] : y[2]), swap_lane8(upper8 ? x[3] : y[3])};
                v = upper8 ? got : x;
            } else {
                v = upper8 ? y : got;
            }
            const uint32_t row = (uint32_t)(pair / 2 * 32 + 8 * (phase - 2)) * 2u * (uint32_t)g.N;
            __builtin_amdgcn_raw_buffer_store_b128(v, d_rsrc, (int)(d_off[pair % 2] + row), 0, 0);
        };
        if constexpr (phase == 0) exchange(blks[0][0], blks[0][1], w00, w10);
        else if constexpr (phase == 1) exchange(blks[1][0], blks[1][1], w01, w11);
        else if constexpr (phase < 4) put(w00, w01);
        else put(w10, w11);
    };
    auto store_pair = [&](int pair, const u32x4 (&blks)[2][2]) {
        for_each_below<6>([&](auto phase) { store_phase(pair, blks, phase); });
    };

    // ---- one k-step, slot by slot (see fine_step of mac_loop): matrix-core instruction (START: accumulators from zero), its
    // share of the reads of the next k-step's operands and of the requests (B in the first half of a trip, A in the second)
    Acc acc[C::MI][C::NI];
    Frags<C> f[2];
    int ca = C::NSA - 1, cb = C::NSB - 1;              // ring slots of the stage before the one handed over (they take the requests)
    unsigned char *a_next, *b_next;                    // the stage handed over
    // Block b of the finished tile leaves the accumulators
    u32x4 at_once[2][2];
    auto take_block = [&](auto number) {
        constexpr int b = decltype(number)::value, pair = b / 2;
        if constexpr (pair < W::KEPT) {
            pack_block(acc[b / C::NI][b % C::NI], out[pair][b % 2]);
        } else {
            pack_block(acc[b / C::NI][b % C::NI], at_once[b % 2]);
            if constexpr (b % 2 == 1) store_pair(pair, at_once);
        }
    };
    auto step = [&](auto pos, auto start, auto last, auto pair, const Frags<C>& cur, Frags<C>& nxt, int kk_next) {
        constexpr int R = Frags<C>::READS, NRS = NM * 3 / 4;
        for_each_below<NM>([&](auto slot) {
            constexpr int s = decltype(slot)::value, mi = s / C::NI, ni = s % C::NI, u = decltype(pos)::value * NM + s;
            acc[mi][ni] = Mfma<C::DT, C::MF>::run(cur.b[ni], cur.a[mi], decltype(start)::value ? Acc{} : acc[mi][ni]);
            if (s < NRS) {
#pragma unroll
                for (int r = s * R / NRS; r < (s + 1) * R / NRS; r++) nxt.load_one(a_next, b_next, fm, kk_next, r);
            }
            requests(u * C::LPS / SLOTS, (u + 1) * C::LPS / SLOTS, ca, cb);
            constexpr int PAIR = decltype(pair)::value;
            if constexpr (decltype(last)::value) __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(last)::value && s >= W::TAKEN_LATE) take_block(std::integral_constant<int, s - W::TAKEN_LATE>());
            constexpr int t = u - SLOTS / 2, EACH = SLOTS / 16;
            if constexpr (PAIR >= 0 && t >= 0 && t % EACH == 0 && t / EACH < 6) store_phase(PAIR, out[PAIR], std::integral_constant<int, t / EACH>());
            __builtin_amdgcn_sched_barrier(0);
        });
        // (or the compiler sinks the whole k-step behind the branch that follows, away from its reads and requests)
#pragma unroll
        for (int s = 0; s < NM; s++) asm volatile("" : "+a"(acc[s / C::NI][s % C::NI]));
    };
    const int tail_trip = full_k < nk ? nk - 2 : nk;   // the trip that hands over a last, ragged k-iteration
    // Hand over stage i + 1: its loads have landed (STORES: issued after its last one, may still be in flight), and all waves
    // are done with the operands of stage i
    auto hand_over = [&](int i, auto stores, bool check) {
        const int na = ca + 1 == C::NSA ? 0 : ca + 1, nb = cb + 1 == C::NSB ? 0 : cb + 1;
        a_next = smem + na * C::A_BYTES;
        b_next = smem + C::B_RING + nb * C::B_BYTES;
        wait_vmcnt<C::A_LD + decltype(stores)::value>();
        __syncthreads();
        if (__builtin_expect(check && i == tail_trip, 0)) {
            if (full_k * C::BK + a_col >= g.K) {
#pragma unroll 1
                for (int j = 0; j < C::A_LD; j++) reinterpret_cast<uint4*>(a_next)[tid + j * C::THREADS] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll 1
            for (int j = (g.K - full_k * C::BK) / B_ROWS; j < C::B_LD; j++) reinterpret_cast<uint4*>(b_next)[tid + j * C::THREADS] = make_uint4(0, 0, 0, 0);
            __syncthreads();
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The k-steps of the handed-over stage but its last; in the second half one pair of the kept blocks leaves
    auto most_steps = [&](auto start, auto pair, bool check) {
        for_each_below<KK - 1>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            step(std::integral_constant<int, k + 1>(), std::integral_constant<bool, decltype(start)::value && k == 0>(), No(), pair, f[k & 1], f[(k + 1) & 1], k + 1);
        });
        ca = ca + 1 == C::NSA ? 0 : ca + 1;
        cb = cb + 1 == C::NSB ? 0 : cb + 1;
        advance_b(check);
        advance_a(check);
    };
    typedef std::integral_constant<int, -1> Nothing;
    typedef std::integral_constant<int, 0> Zero;
    auto trip = [&](int i, auto pair, auto stores, bool check) {
        hand_over(i, stores, check);
        step(Zero(), No(), No(), pair, f[1], f[0], 0);
        most_steps(No(), pair, check);
    };

    // ---- first requests (a trip's order: B of stage s, A of stage s + 1) and the first stage's first operands
    map_a(m0);
    map_b(n0);
    requests(C::B_LD, C::LPS, 0, 0);
    advance_a(false);
    requests(0, C::LPS, 1, 0);
    advance_b(false);
    advance_a(false);
    hand_over(-1, Zero(), false);
    f[0].load(a_next, b_next, fm, 0);
    requests(0, C::LPS / KK, ca, cb);
    __builtin_amdgcn_sched_barrier(0);
    most_steps(Yes(), Nothing(), false);
    int i = 0;
    while (true) {
        for (; i < nk - W::CHECKED; i++) trip(i, Nothing(), Zero(), false);
        for (; i < nk - 1; i++) trip(i, Nothing(), Zero(), true);
        aim();
        hand_over(nk - 1, Zero(), false);
        step(Zero(), No(), Yes(), Nothing(), f[1], f[0], 0);
        // the turn: the tile's last k-step is done, with the requests and reads of the next tile's first; its blocks are packed
        for_each_below<W::TAKEN_LATE>([&](auto b) {
            take_block(std::integral_constant<int, NM - W::TAKEN_LATE + decltype(b)::value>());
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!more) break;
        m0 = m0_next;
        n0 = n0_next;
        more = next_tile(m0_next, n0_next);
        most_steps(Yes(), Zero(), false);
        for_each_below<W::KEPT - 1>([&](auto p) {
            constexpr int n = decltype(p)::value;
            trip(n, std::integral_constant<int, n + 1>(), std::integral_constant<int, W::PAIR_STORES * (n == 0 ? W::after_requests() + 1 : 1)>(), n >= nk - W::CHECKED);
        });
        i = W::KEPT - 1;
    }
    // the last tile's blocks leave as they lie, 32 rows of 32 bytes per store: there is no matrix-core work beside an exchange
    const uint32_t first = ((uint32_t)(wm * C::WTM + lane % 32) * (uint32_t)g.N + (uint32_t)(wn * C::WTN + 8 * (lane / 32))) * 2u;
    for_each_below<2 * W::KEPT>([&](auto number) {
        constexpr int b = decltype(number)::value, mi = b / C::NI, ni = b % C::NI;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const bool inside = n0 + wn * C::WTN + 8 * (lane / 32) + ni * 32 + 16 * h < g.N;
            __builtin_amdgcn_raw_buffer_store_b128(out[b / 2][b % 2][h], d_rsrc, (int)(inside ? first + mi * 64 * (uint32_t)g.N + (ni * 64 + 32 * h) : 0x80000000u), 0, 0);
        }
    });
    // the requests beyond the last tile have landed before the workgroup's LDS goes to another one
    wait_vmcnt<W::PAIR_STORES * (W::KEPT + W::after_requests())>();
}

template <class C>
__global__ __launch_bounds__(C::THREADS) void streamk_whole_tiles_kernel(GemmArgs g) {
    extern __shared__ __align__(1024) unsigned char smem[];
    if (g.out_dtype == SK_BF16) whole_tiles<C, SK_BF16>(g, smem);
    else whole_tiles<C, SK_F16>(g, smem);
}

// The entry of C's own four-wave kernel gets it.
template <class C> void add_across(KernelEntry** t, int n) {
    for (int i = 0; i < n; i++)
        if (t[i]->dtype == C::DT && t[i]->bm == C::BM && t[i]->bn == C::BN && t[i]->bk == C::BK && t[i]->threads == C::THREADS && t[i]->fixup == SK_FIXUP_FLAGS) {
            t[i]->across = streamk_whole_tiles_kernel<C>;
            t[i]->across_iters = WholeTiles<C>::MIN_ITERS;
        }
}

}  // namespace streamk_detail
