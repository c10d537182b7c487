// The loop over the items of a workgroup: the body of batch_kernel and of
// batch_body, as text, since the compiler makes different code of the two
// (see batch_body).  In scope: B and the template arguments SCHEME, CPT, COLS, FL,
// LD, NW and LANES.
    constexpr bool SHARED = LD > 0 || NW > 0;
    extern __shared__ uint32_t smem[];
    // lattice, tile, generation, stop; the neighbourhood to wait for: first
    // column, columns, first row, rows
    __shared__ uint32_t cmd[8];
    const uint32_t tid = threadIdx.x;
    uint32_t my_stamp = 0;
    for (;;) {
        if (tid < 64u) {
            if (tid == 0) {
                uint32_t r = 0, t = 0, g = 0, stop = 0;
                uint32_t cx0 = 0, ncol = 0, cy0 = 0, nrow = 0;
                const unsigned long long i = atomicAdd(B.ticket, 1ull);
                if (i >= B.total_items || __hip_atomic_load(B.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    stop = 1;
                } else {
                    uint32_t lo = 0, hi = B.nphase;
                    while (hi - lo > 1u) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (B.phases[mid].first_item <= i) lo = mid; else hi = mid;
                    }
                    const BatchPhase ph = B.phases[lo];
                    const uint64_t rel = i - ph.first_item;
                    g = ph.gen_begin + (uint32_t)(rel / ph.items_per_gen);
                    const uint32_t off = (uint32_t)(rel % ph.items_per_gen);
                    lo = 0;
                    hi = ph.nslots;
                    while (hi - lo > 1u) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (B.tile_prefix[mid] <= off) lo = mid; else hi = mid;
                    }
                    r = lo;
                    t = off - B.tile_prefix[r];
                    if (g > 0u) {
                        // the tiles of generation g - 1 whose words this item can share
                        const BatchSlot &S = B.slots[r];
                        const bool new_tiling = (g & 3u) == 0u;
                        uint32_t ox = 0, oy = 0, oxp = 0, oyp = 0;
                        if (new_tiling) {
                            const uint64_t m = B.mcs_base[r] + (g >> 2);
                            (void)mcs_origin(S, m, ox, oy);
                            (void)mcs_origin(S, m - 1u, oxp, oyp);
                        }
                        const WaitSet ws = wait_set(S.a.Dx, S.a.Dy, S.a.L_mask, S.a.log2ntx, S.ntiles, t,
                                                    new_tiling, ox, oy, oxp, oyp);
                        cx0 = ws.cx0;
                        ncol = ws.ncol;
                        cy0 = ws.cy0;
                        nrow = ws.nrow;
                    }
                }
                cmd[0] = r;
                cmd[1] = t;
                cmd[2] = g;
                cmd[3] = stop;
                cmd[4] = cx0;
                cmd[5] = ncol;
                cmd[6] = cy0;
                cmd[7] = nrow;
                my_stamp = stop ? 0u : B.tile_prefix[r] + t;
            }
            wave_order();
            // The first wave waits for the neighbourhood, one stamp per lane (and
            // for tile t itself, so that each tile finishes its generations in
            // order and its stamp counts them), every wait bounded in time.
            const uint32_t g = cmd[2];
            if (!cmd[3] && g > 0u) {
                const uint32_t r = cmd[0], t = cmd[1], cx0 = cmd[4], ncol = cmd[5], cy0 = cmd[6], nrow = cmd[7];
                const BatchSlot &S = B.slots[r];
                const uint32_t lx = S.a.log2ntx, ntx = 1u << lx, nty = S.ntiles >> lx;
                const uint32_t *st = B.stamp + B.tile_prefix[r];
                const uint32_t nwait = ncol * nrow + 1u;
                const uint64_t t0 = wall_clock64();
                bool bad = false;
                for (uint32_t nb = tid; nb < nwait; nb += 64u) {
                    const uint32_t nx = (cx0 + nb % ncol) & (ntx - 1u);
                    const uint32_t ny = (cy0 + nb / ncol) & (nty - 1u);
                    const uint32_t *sp = nb + 1u < nwait ? st + ((ny << lx) | nx) : st + t;
                    while (!bad && __hip_atomic_load(sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < g) {
                        if (__hip_atomic_load(B.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                            bad = true;
                        } else if (wall_clock64() - t0 > B.wait_ticks) {
                            atomicOr(B.error, 1u);
                            bad = true;
                        } else {
                            __builtin_amdgcn_s_sleep(2);
                        }
                    }
                }
                const uint64_t any_bad = __ballot(bad);  // every lane of the wave takes part
                // generic sweeps read through the caches: the earlier steps' words, written by
                // other workgroups, become visible (the invalidation covers the whole
                // workgroup's caches)
                if (!SHARED) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                if (tid == 0 && any_bad) cmd[3] = 1u;
            }
        }
        __syncthreads();
        if (cmd[3]) break;
        const uint32_t r = __builtin_amdgcn_readfirstlane(cmd[0]);
        const uint32_t tile = __builtin_amdgcn_readfirstlane(cmd[1]);
        const uint32_t g = __builtin_amdgcn_readfirstlane(cmd[2]);
        const BatchSlot &S = B.slots[r];
        StepArgs A = SHARED ? uniform(S.a) : S.a;
        // MCS draw of the lattice's MCS m (as on the host): origin and set order
        const uint64_t m = B.mcs_base[r] + (g >> 2);
        const uint32_t k = g & 3u;
        uint32_t ox, oy;
        const u32x4 w = mcs_origin(S, m, ox, oy);
        const uint32_t set = perm_element((uint32_t)(((uint64_t)w.z * 24u) >> 32), k);
        A.ox = ox;
        A.oy = oy;
        A.set_a = set & 1u;
        A.set_b = set >> 1;
        A.c3 = (uint32_t)(m << 2) | k;
        // Visibility of the earlier steps' words, written by other workgroups.
        // Generic sweeps: the first wave took the agent-scope acquire after its
        // waits, before the barrier above (it invalidates the caches this
        // workgroup reads through, which all its waves share).  SHARED sweeps:
        // no acquire; every load and store of lattice words in them is an
        // agent-scope atomic (load_word, load_words, store_words), which goes to
        // where all dies see it, and is issued after the barrier, so after the
        // stamps were seen.  A plain access to lattice words in a SHARED sweep
        // would break this.
        if constexpr (NW > 0) {
            const bool draws = S.accept != 0u;
            if constexpr (NW == 1) {
                batch_dt_cells<7, NW>(A, smem, tile, draws);
            } else if constexpr (NW == 2) {
                if (A.Dx == 128u)
                    batch_dt_cells<7, NW>(A, smem, tile, draws);
                else
                    batch_dt_cells<8, NW>(A, smem, tile, draws);
            } else {
                batch_dt_cells<8, NW>(A, smem, tile, draws);
            }
        } else if constexpr (SCHEME == kDB && LD > 0 && CPT == 1) {
            sweep_db_cells<FL == 4, LD, true>(A, smem, tile);
        } else if constexpr (LD > 0 && SCHEME != kDB) {
            if (A.Dx == 256u) {
                if (S.accept)
                    sweep_dt_rows<SCHEME, true, CPT, 8, 3, true>(A, smem, tile);
                else
                    sweep_dt_rows<SCHEME, false, CPT, 8, 3, true>(A, smem, tile);
            } else {
                if (S.accept)
                    sweep_dt_rows<SCHEME, true, CPT, 7, 3, true>(A, smem, tile);
                else
                    sweep_dt_rows<SCHEME, false, CPT, 7, 3, true>(A, smem, tile);
            }
        } else if constexpr (LD > 0) {
            sweep_db_rows<FL == 4, CPT, LD, 3, true>(A, smem, tile);
        } else if constexpr (COLS && FL > 0) {
            sweep_db_columns<FL == 4, CPT, FL>(A, smem, tile);
        } else if constexpr (COLS) {
            if (S.accept)
                sweep_db_columns<true, CPT, 0>(A, smem, tile);
            else
                sweep_db_columns<false, CPT, 0>(A, smem, tile);
        } else {
            if (S.accept)
                sweep_tile<SCHEME, true, CPT, false, LANES>(A, smem, tile);
            else
                sweep_tile<SCHEME, false, CPT, false, LANES && CPT == 2>(A, smem, tile);
        }
        // Publish this tile's words before stamping the tile with generation g
        // done: every lane waits until its own stores are acknowledged and the
        // barrier orders them before thread 0's stamp.  Generic sweeps: the stamp
        // is an agent-scope release store, which writes the words back for the
        // other dies (once per item, not once per wave).  SHARED sweeps: the
        // acknowledged stores are there already and the stamp is relaxed; the
        // fence of one thread, no instruction, keeps the compiler from moving
        // them past the wait.
        if (SHARED) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "singlethread");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0)
            __hip_atomic_store(&B.stamp[my_stamp], g + 1u, SHARED ? __ATOMIC_RELAXED : __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
