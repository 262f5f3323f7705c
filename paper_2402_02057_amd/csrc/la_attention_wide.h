// Lookahead-step attention for batches of many rows (included by la_attention.hip, whose parameters,
// chunks, swizzle, masks and arithmetic it shares; head_dim 128, packed or paged bf16 caches): workgroups
// of up to 256 rows whose waves take turns on the matrix cores.
//
// What bounds the staged kernel here: its 128-row workgroups take 1.14 to 1.22 us per 64-key chunk, of which the
// matrix cores need 0.44.  The two waves of a SIMD leave a barrier together and do the same things at
// the same time, so scores, softmax and PV follow each other instead of overlapping; and with four row
// tiles a chunk is staged, and a barrier passed, for only half of this kernel's work.
//
// A wave owns one 32-row tile and walks all keys of its workgroup's range: eight tiles share a chunk.  Waves
// 4 .. 7 (w and w + 4 share a SIMD) run half a period behind: between two barriers the early wave does
// its matrix phase (PV of the last chunk, scores of this one: 36 products whose operands are read a batch
// ahead) and then its softmax, the late one its softmax and then its matrix phase, on the same data.
// K of a chunk is read in its own period, V in the next, so a stage is free two barriers after its
// chunk arrived; five stages of 32 KB leave three chunks in flight.  The query rows pass through the two
// stages that are requested last.  Nothing is merged between waves, and no sum is rounded to bf16.
//
// A range of a cut step leaves its rows in fp32 (unnormalised, with maximum and sum); wide_combine_kernel
// adds the ranges up, in index order.  (The staged kernel's exchange inside the launch was tried: the
// workgroup that arrives last pulls 132 KB per range through one compute unit, 15 us for four ranges; a
// kernel of its own spreads that over the GPU, 6 us with its launch.)
//
// Measured (us a launch in a graph, staged and here): 8 x 1024 keys, 64/8 heads, 121 rows 61 and 50; 8 x 3072 keys
// 139 and 108 (1.81 us a chunk of 256 rows, 2.3 staged); 8 x 1024 keys, 128/32 heads, 61 rows 63 and 47; 8
// prefixes of 1253 to 14559 keys, 32/8 heads, 121 rows 158 and 134; 16 of 466 to 1021 keys, 81 rows 44 and 38.
// Pages cost nothing here: the ragged eight take 132 to 135 packed, on pages of 64 or 256 keys, shuffled or in order.
// Relative error against 64 bits, staged and here: 2.66e-3 and 2.33e-3 for the ragged eight, 2.71e-3 and 2.31e-3 for the sixteen.
// What bounds it now is power: with random operands 32x32x16 products alone run at 2.0 GHz, with a
// block's softmax and operand reads beside them at 1.8 (3160 cycles a chunk, 2100 of them products).
// Tried and dropped: one wave per SIMD with two tiles (half the operand reads; products, exponentials and
// reads interleaved one by one, 390 registers, no copies): 4190 cycles a chunk at 2.2 GHz, 1.9 us, as a lone
// wave waits out its own requests; 128-row workgroups of this kind: as fast as the staged ones.
#pragma once

struct WideCfg {
    static constexpr int HEAD_DIM = 128, KC = 64, NSTAGE = 5;
    static constexpr int NW = 8, NT = NW * 64, TILES = NW;  // a wave has a 32-row tile and walks all keys of the range
    static constexpr int RBYTES = HEAD_DIM * 2, KV_BYTES = KC * RBYTES, STAGE_BYTES = 2 * KV_BYTES;
    static constexpr int LPW = STAGE_BYTES / 1024 / NW;     // loads per wave and chunk
    static constexpr int AHEAD = NSTAGE - 2;                // chunks requested ahead of the one being read
    static constexpr int Q_OFFSET = AHEAD * STAGE_BYTES;    // the query rows land in the stages not requested yet
    static constexpr int QLPW = TILES * 32 * RBYTES / 1024 / NW;
    static_assert(TILES * 32 * RBYTES <= 2 * STAGE_BYTES, "the query rows fit the last two stages");
    static constexpr int DB = HEAD_DIM / 32;
    // partial results, per wave: its tile in fp32 and fragment order, then (m, l) of its rows
    static constexpr int PART_ACC_BYTES = DB * 16 * 64 * 4;
    static constexpr int PART_WAVE_BYTES = PART_ACC_BYTES + 64 * 8;
    static constexpr int PART_WG_BYTES = NW * PART_WAVE_BYTES;
    static constexpr int COMBINE_WGS = NW * DB / 4;         // workgroups of four waves that add up a row block's ranges
    static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
};

#define SB() __builtin_amdgcn_sched_barrier(0)
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// A wave's finished tile goes to `out` through its own 8 KB of LDS: from registers a store covers 16 bytes of
// each of 32 rows, turned around it covers whole rows of 256 (a workgroup's rows: 3.5 -> 1.2 us after the
// loop).  16-byte pieces of a row are stored XORed with the row, so that neither side has bank conflicts.
template <class C>
__device__ __forceinline__ void stage_slice(unsigned char* stage, int lane, int u, const f32x16& vals, float inv)
{
    constexpr int PIECES = C::DB * 4;   // of a row
    const int l32 = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (__bf16)(vals[i4 * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(stage + l32 * (PIECES * 16) + (((u * 4 + i4) ^ (l32 & (PIECES - 1))) << 4) + hi * 8) = v;
    }
}
template <class C>
__device__ __forceinline__ void store_rows(const AttnParams& p, const unsigned char* stage, int row_base, int kvh, int lane)
{
    constexpr int PIECES = C::DB * 4;
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += 64 / PIECES) {
        const int row = r0 + lane / PIECES, piece = lane % PIECES;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + row * (PIECES * 16) + ((piece ^ (row & (PIECES - 1))) << 4));
        const int rr = row_base + row;
        if (rr < p.R) {
            const int t = div_small(rr, p.inv_group), hh = rr - t * p.group;
            *reinterpret_cast<bf16x8*>(p.out + ((size_t)t * p.heads + (size_t)kvh * p.group + hh) * C::HEAD_DIM + piece * 8) = v;
        }
    }
}

template <bool PAGED>
__device__ __forceinline__ void wide_attention_body(const AttnParams& p, const int xcd, const int slot)
{
    using C = WideCfg;
    constexpr int D = C::HEAD_DIM, KC = C::KC, NSTAGE = C::NSTAGE;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int logical = xcd * p.wg_per_xcd + slot;
    if (logical >= p.total_wg) return;
    const int unit = __builtin_amdgcn_readfirstlane(div_small(logical, p.inv_XS));
    const int xs = logical - unit * p.XS;
    const int kvh = __builtin_amdgcn_readfirstlane(div_small(unit, p.inv_row_blocks));
    const int rb = unit - kvh * p.n_row_blocks;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hi = lane >> 5, l32 = lane & 31;
    const bool late = wave >= C::NW / 2;   // waves w and w + 4 share a SIMD
    const unsigned lds_base = lds_address(lds);
    const int row_base = rb * p.block_rows + wave * 32;
    const bool wave_active = wave * 32 < p.block_rows && row_base < p.R;

    const int c_begin = xs * p.chunks_lo + min(xs, p.chunks_rem);
    const int n_my = p.chunks_lo + (xs < p.chunks_rem ? 1 : 0);

    // ---- requests
    static_assert(C::LPW == 4, "a wave fetches two groups of four rows, 32 rows apart, of K and of V");
    const int ld_row = wave * 4 + (lane >> 4);
    const unsigned ld_piece = (unsigned)(((lane & 15) ^ swizzle<D>(ld_row)) << 4);  // (the same 32 rows on)
    const unsigned ld_off = (unsigned)(ld_row * C::RBYTES) + ld_piece;
    const unsigned char* const kc_head = reinterpret_cast<const unsigned char*>(p.k_cache) + (size_t)kvh * (size_t)p.cache_rows * C::RBYTES;
    const unsigned char* const vc_head = reinterpret_cast<const unsigned char*>(p.v_cache) + (size_t)kvh * (size_t)p.cache_rows * C::RBYTES;
    const unsigned char* const sk_head = reinterpret_cast<const unsigned char*>(p.step_k) + (size_t)kvh * C::RBYTES;
    const unsigned char* const sv_head = reinterpret_cast<const unsigned char*>(p.step_v) + (size_t)kvh * C::RBYTES;
    const unsigned step_stride = (unsigned)(p.kv_heads * C::RBYTES);
    const int n_prefix_chunks = p.n_prefix_chunks, n_P = p.P, n_T = p.T;

    const unsigned char* iss_k;
    const unsigned char* iss_v;
    int iss_c;                    // next chunk to request
    unsigned iss_stage;
    // Paged cache: lane i holds the table entry of page pg_base + i.  Entries are loaded 64 at a time, with
    // their wait in the same statement: the compiler's own wait stood in front of every use, once a page, and a wait
    // for a vector load is one for all chunks in flight (the ragged eight, pages of 64 keys 149 -> 134 us a layer, of 256 141 -> 135).
    int pg_base = 0, pg_ents = 0, iss_page = 0, iss_page_left = 0;
    const int page_last = PAGED ? p.n_pages - 1 : 0;
    const size_t page_bytes = PAGED ? (size_t)p.page_bytes : 0;
    auto load_entries = [&](int first) {
        pg_base = first;
        // (five wait states, in case the pointer was written by the vector unit just now: see `dma16_base`)
        asm volatile("s_nop 4\n\tglobal_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)"
                     : "=&v"(pg_ents)
                     : "v"((unsigned)min(first + lane, p.table_last) * 4u), "s"(p.block_table)
                     : "memory");
    };
    auto page_base = [&]() {
        if (iss_page - pg_base >= 64) load_entries(iss_page);
        const int raw = __builtin_amdgcn_readlane(pg_ents, iss_page - pg_base);
        return (size_t)min(max(raw, 0), page_last) * page_bytes;
    };
    auto seek = [&](int c) {
        iss_c = c;
        iss_stage = 0;
        if (c < n_prefix_chunks) {
            size_t off = (size_t)c * (KC * C::RBYTES);
            if constexpr (PAGED) {
                iss_page = __builtin_amdgcn_readfirstlane(div_small(c, p.inv_page_chunks));
                const int within = c - iss_page * p.page_chunks;
                load_entries(iss_page);
                iss_page_left = p.page_chunks - within;
                off = page_base() + (size_t)within * (KC * C::RBYTES);
            }
            iss_k = kc_head + off;
            iss_v = vc_head + off;
        } else {
            const size_t off = (size_t)(c - n_prefix_chunks) * KC * step_stride;
            iss_k = sk_head + off;
            iss_v = sv_head + off;
        }
    };
    auto issue_next = [&]() {
        const unsigned dst = lds_base + iss_stage + (unsigned)wave * 1024u;
        const int c = iss_c++;
        const bool step = c >= n_prefix_chunks;
        const int rows = step ? n_T - (c - n_prefix_chunks) * KC : n_P - c * KC;
        unsigned off0 = ld_off, off1 = ld_off + 32 * C::RBYTES;
        if (step || rows < KC) {
            const int last_row = min(KC, rows) - 1;
            const unsigned stride = step ? step_stride : (unsigned)C::RBYTES;
            int row = lane;
            asm volatile("" : "+v"(row));
            row = wave * 4 + (row >> 4);
            off0 = __umul24((unsigned)min(row, last_row), stride) + ld_piece;
            off1 = __umul24((unsigned)min(row + 32, last_row), stride) + ld_piece;
        }
        dma16_base(iss_k, off0, dst);
        dma16_base(iss_v, off0, dst + C::KV_BYTES);
        dma16_base(iss_k, off1, dst + 8 * 1024);
        dma16_base(iss_v, off1, dst + C::KV_BYTES + 8 * 1024);
        iss_stage = iss_stage + C::STAGE_BYTES == (unsigned)(NSTAGE * C::STAGE_BYTES) ? 0u : iss_stage + C::STAGE_BYTES;
        if (iss_c >= n_prefix_chunks) {
            const size_t o = (size_t)(iss_c - n_prefix_chunks) * KC * step_stride;
            iss_k = sk_head + o;
            iss_v = sv_head + o;
        } else if (PAGED && --iss_page_left == 0) {
            ++iss_page;
            iss_page_left = p.page_chunks;
            const size_t o = page_base();
            iss_k = kc_head + o;
            iss_v = vc_head + o;
        } else {
            iss_k += KC * C::RBYTES;
            iss_v += KC * C::RBYTES;
        }
    };
    auto issue_q = [&]() {
#pragma unroll
        for (int i = 0; i < C::QLPW; ++i) {
            const int wl = wave + i * C::NW;
            if (wl * 4 >= p.block_rows) continue;
            const int row = wl * 4 + (lane >> 4);
            const int lc = (lane & 15) ^ swizzle<D>(row);
            const int rr = min(rb * p.block_rows + row, p.R - 1);
            const int t = div_small(rr, p.inv_group), hh = rr - t * p.group;
            dma16_base(p.q, (unsigned)(((t * p.heads + kvh * p.group + hh) * D + lc * 8) * 2), lds_base + C::Q_OFFSET + wl * 1024);
        }
    };

    int issued = 0;
    seek(c_begin);
    issue_next();
    issue_q();
    issued = min(n_my, C::AHEAD);
#pragma unroll
    for (int s = 1; s < C::AHEAD; ++s)
        if (s < issued) issue_next();

    const int t_lane = div_small(min(row_base + l32, p.R - 1), p.inv_group);
    const float sl2 = p.scale_log2;
    bf16x8 qreg[D / 16];
    f32x16 o[C::DB];
    float m_run, l_run;
    f32x4 lsum;
    const bf16x8 pick = row_sum_operand(lane);

    // LDS addresses of the reads in stage 0.  Piece and column of a read are XORed in as it is made (address
    // bits 5 to 7, which the swizzle leaves as a plain XOR): fifteen registers less than an address each.
    unsigned k_base, v_base;
    {
        const int krow = l32;
        k_base = lds_base + (unsigned)(krow * C::RBYTES + ((hi ^ swizzle<D>(krow)) << 4));
        const int b16 = lane >> 4, i16 = lane & 15, jj = i16 >> 2, q4 = i16 & 3;
        const int vrow = hi * 4 + jj;
        v_base = lds_base + (unsigned)(C::KV_BYTES + vrow * C::RBYTES + ((((b16 & 1) * 2 + (q4 >> 1)) ^ swizzle<D>(vrow)) << 4) + (q4 & 1) * 8);
    }
    typedef const __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    typedef __attribute__((address_space(3))) short4v lds_short4;
    m_run = kNegInf;
    l_run = 0.0f;
    lsum = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.0f;
    wait_young<C::LPW, C::AHEAD - 1>(issued - 1);
    wg_barrier();
    const int qrow = wave * 32 + l32;
    const unsigned char* qr = lds + C::Q_OFFSET + qrow * C::RBYTES;
    const int qsw = swizzle<D>(qrow);
#pragma unroll
    for (int k16 = 0; k16 < D / 16; ++k16)
        qreg[k16] = *reinterpret_cast<const bf16x8*>(qr + (((k16 * 2 + hi) ^ qsw) << 4));
    asm volatile("s_waitcnt lgkmcnt(0)" ::"v"(qreg[0]), "v"(qreg[1]), "v"(qreg[2]), "v"(qreg[3]), "v"(qreg[4]), "v"(qreg[5]), "v"(qreg[6]), "v"(qreg[7]) : "memory");
    wg_barrier();

    // state between the phases of a wave
    f32x16 s[2];
    bf16x8 pf[2][2];
    bf16x8 opA[8], opB[8];

    // chunk j is complete in LDS, and everyone is through with the scores of chunk j-1 and the values of j-2
    auto arrive = [&](int j) {
        wait_young<C::LPW, C::AHEAD - 1>(issued - (j + 1));
        wg_barrier();
    };
    auto request = [&]() {
        if (issued < n_my) {
            issue_next();
            ++issued;
        }
    };
    auto read_k = [&](bf16x8& dst, unsigned at, int b, int k16) {
        dst = *((lds_bf16x8*)(size_t)(at ^ (unsigned)(k16 << 5)) + b * 32 * (C::RBYTES / 16));
    };
    auto read_v = [&](bf16x8& dst, unsigned at, int b, int kk, int db) {
        union { struct { short4v a, b; } s; bf16x8 v; } u;
        u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(size_t)(at ^ (unsigned)(db << 6)) + (b * 32 + kk * 16) * (C::RBYTES / 8));
        u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(size_t)(at ^ (unsigned)((db << 6) | 32)) + (b * 32 + kk * 16 + 8) * (C::RBYTES / 8));
        dst = u.v;
    };
    auto pv = [&](const bf16x8& v, int b, int kk, int db) {
        if (db == 0) lsum = add_row_sums(pick, pf[b][kk], lsum);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pf[b][kk], o[db], 0, 0, 0);
    };
    auto qk = [&](const bf16x8& k, int b, int k16) {
        if (k16 == 0)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[b][i] = 0.0f;
        s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, qreg[k16], s[b], 0, 0, 0);
    };
    // The first `nb` blocks of s become weights in pf; reference and accumulators move with them as in the staged kernel.
    auto softmax = [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
#pragma unroll
        for (int b = 0; b < NB; ++b) settle_mfma_result(s[b]);
        float mx[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            mx[b] = max3(s[b][0], s[b][1], s[b][2]);
#pragma unroll
            for (int i = 3; i < 15; i += 2) mx[b] = max3(mx[b], s[b][i], s[b][i + 1]);
        }
        const float m_blk = max_across_halves(NB == 2 ? max2(max3(mx[0], s[0][15], mx[NB - 1]), s[NB - 1][15]) : max2(mx[0], s[0][15]));
        const bool move = reference_moves(m_blk, m_run, sl2);
        const float m_new = move ? m_blk : m_run;
        const float m_use = (m_new == kNegInf) ? 0.0f : m_new;  // the row has seen no key at all
        const float bias = weight_bias(m_use, sl2);
        if (__builtin_amdgcn_ballot_w64(move) != 0ull) {
            const float alpha = moved_by(m_run, m_use, sl2);
            scale_row_sums(lsum, alpha, lane);
#pragma unroll
            for (int db = 0; db < C::DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
        }
        m_run = m_new;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) pf[b][i >> 3][i & 7] = (__bf16)weight(s[b][i], sl2, bias);
    };
    constexpr std::integral_constant<int, 1> one;
    constexpr std::integral_constant<int, 2> both;
    auto next_stage = [&](unsigned st) {
        return st + C::STAGE_BYTES == (unsigned)(NSTAGE * C::STAGE_BYTES) ? 0u : st + C::STAGE_BYTES;
    };

    if (!wave_active) {   // only helps loading
        for (int j = 0; j < n_my; ++j) {
            if (j > 0) arrive(j);
            request();
        }
    } else {
        unsigned stage = 0;
        // ---- the chunks of 64 prefix keys, which every row sees
        const int n_full = min(n_my, n_P / KC - c_begin);
        if (n_full > 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) read_k(opA[i], k_base, i & 1, i >> 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) { qk(opA[i], i & 1, i >> 1); read_k(opB[i], k_base, i & 1, 4 + (i >> 1)); }
#pragma unroll
            for (int i = 0; i < 8; ++i) { qk(opB[i], i & 1, 4 + (i >> 1)); read_v(opA[i], v_base, 0, i >> 2, i & 3); }
            for (int j = 1; j < n_full; ++j) {
                if (late) arrive(j);
                request();
                softmax(both);
                if (!late) arrive(j);
                // Matrix phase: PV of the previous chunk, then the scores of this one.  Operands are read a batch
                // of eight products ahead, each read behind a product: requested in front of a batch they
                // leave the matrix cores idle until LDS has taken them all (2.03 -> 1.81 us a chunk).
                const unsigned next = next_stage(stage), k_at = k_base + next, v_at = v_base + stage, v_next = v_base + next;
                SB();
#pragma unroll
                for (int i = 0; i < 8; ++i) { pv(opA[i], 0, i >> 2, i & 3); read_v(opB[i], v_at, 1, i >> 2, i & 3); SB(); }
#pragma unroll
                for (int i = 0; i < 8; ++i) { pv(opB[i], 1, i >> 2, i & 3); read_k(opA[i], k_at, i & 1, i >> 1); SB(); }
#pragma unroll
                for (int i = 0; i < 8; ++i) { qk(opA[i], i & 1, i >> 1); read_k(opB[i], k_at, i & 1, 4 + (i >> 1)); SB(); }
#pragma unroll
                for (int i = 0; i < 8; ++i) { qk(opB[i], i & 1, 4 + (i >> 1)); read_v(opA[i], v_next, 0, i >> 2, i & 3); SB(); }
                stage = next;
            }
            softmax(both);
            const unsigned v_at = v_base + stage;
#pragma unroll
            for (int i = 0; i < 8; ++i) { pv(opA[i], 0, i >> 2, i & 3); read_v(opB[i], v_at, 1, i >> 2, i & 3); }
#pragma unroll
            for (int i = 0; i < 8; ++i) pv(opB[i], 1, i >> 2, i & 3);
            stage = next_stage(stage);
        }
        // ---- the others, block by block under the mask; a block that no row of the tile sees is passed over
        //      before it is read, as wide windows leave many such blocks
        const RowVis vis = row_visibility(t_lane, p.W, p.N, p.inv_W, p.inv_n1);
        for (int j = max(n_full, 0); j < n_my; ++j) {
            if (j > 0) arrive(j);
            request();
            const int c = c_begin + j;
            const bool is_step = c >= n_prefix_chunks;
            const int key0 = (c - (is_step ? n_prefix_chunks : 0)) * KC;
#pragma unroll 1
            for (int b = 0; b < 2; ++b) {
                const int k0 = key0 + b * 32, left = n_P - k0;
                unsigned word = is_step ? step_block_word(vis, k0) : left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u;
                word = (word >> (hi * 4)) & 0x0F0F0F0Fu;
                if (__builtin_amdgcn_ballot_w64(word != 0u) == 0ull) continue;
                const unsigned at = stage + (unsigned)(b * 32 * C::RBYTES);
#pragma unroll
                for (int i = 0; i < 8; ++i) read_k(opA[i], k_base + at, 0, i);
#pragma unroll
                for (int i = 0; i < 8; ++i) { qk(opA[i], 0, i); read_v(opB[i], v_base + at, 0, i >> 2, i & 3); }
                mask_scores(s[0], word);
                softmax(one);
#pragma unroll
                for (int i = 0; i < 8; ++i) pv(opB[i], 0, i >> 2, i & 3);
            }
            stage = next_stage(stage);
        }
    }

    l_run = row_sum(lsum, lane);
    __syncthreads();  // everyone is through with the ring
    if (!wave_active) return;
    if (p.XS == 1) {
        unsigned char* const stage = lds + wave * 8192;
        const float inv = 1.0f / l_run;
#pragma unroll
        for (int u = 0; u < C::DB; ++u) stage_slice<C>(stage, lane, u, o[u], inv);
        store_rows<C>(p, stage, row_base, kvh, lane);
        return;
    }
    // a range of the keys: what wide_combine_kernel adds up, in fp32 and fragment order
    unsigned char* const dst = reinterpret_cast<unsigned char*>(p.partials) +
                               ((size_t)unit * p.XS + xs) * C::PART_WG_BYTES + (size_t)wave * C::PART_WAVE_BYTES;
#pragma unroll
    for (int u = 0; u < C::DB; ++u)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            *reinterpret_cast<f32x4*>(dst + ((u * 4 + i4) * 64 + lane) * 16) =
                f32x4{o[u][i4 * 4], o[u][i4 * 4 + 1], o[u][i4 * 4 + 2], o[u][i4 * 4 + 3]};
    *reinterpret_cast<f32x2*>(dst + C::PART_ACC_BYTES + lane * 8) = f32x2{m_run, l_run};
}

// The ranges of one (32 rows, 32 columns) slice, one wave each, added up in index order: job `job` of
// unit `unit`.  Four ranges a trip.
__device__ __forceinline__ void wide_combine_body(const AttnParams& p, const int unit, const int job)
{
    using C = WideCfg;
    const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = job / C::DB, u = job % C::DB;      // the wave of the workgroups that left it
    const int kvh = __builtin_amdgcn_readfirstlane(div_small(unit, p.inv_row_blocks));
    const int rb = unit - kvh * p.n_row_blocks;
    const int row_base = rb * p.block_rows + wave * 32;
    if (wave * 32 >= p.block_rows || row_base >= p.R) return;
    const unsigned char* const src = reinterpret_cast<const unsigned char*>(p.partials) +
                                     (size_t)unit * p.XS * C::PART_WG_BYTES + (size_t)wave * C::PART_WAVE_BYTES;
    constexpr int MB = 4;
    float m_acc = kNegInf, l_acc = 0.0f;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    for (int s0 = 0; s0 < p.XS; s0 += MB) {
        f32x2 ml[MB];
        f32x4 v[MB][4];
#pragma unroll
        for (int w = 0; w < MB; ++w) {
            const unsigned char* at = src + (size_t)min(s0 + w, p.XS - 1) * C::PART_WG_BYTES;
            ml[w] = *reinterpret_cast<const f32x2*>(at + C::PART_ACC_BYTES + lane * 8);
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) v[w][i4] = *reinterpret_cast<const f32x4*>(at + ((u * 4 + i4) * 64 + lane) * 16);
        }
        float m = m_acc;
#pragma unroll
        for (int w = 0; w < MB; ++w) m = fmaxf(m, ml[w][0]);
        const float m_use = m == kNegInf ? 0.0f : m;      // (no range so far held a key that the row sees)
        const float a0 = fast_exp2((m_acc - m_use) * p.scale_log2);
        m_acc = m;
        l_acc *= a0;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] *= a0;
#pragma unroll
        for (int w = 0; w < MB; ++w) {
            const float a = s0 + w < p.XS ? fast_exp2((ml[w][0] - m_use) * p.scale_log2) : 0.0f;
            l_acc = __builtin_fmaf(ml[w][1], a, l_acc);
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = __builtin_fmaf(v[w][i >> 2][i & 3], a, acc[i]);
        }
    }
    store_slice<C>(p, row_base, kvh, u, l32, hi, acc, 1.0f / l_acc);
}
