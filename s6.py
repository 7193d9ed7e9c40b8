import sys; sys.path.insert(0,'/root/repo/_work/exp')
from sw import mk,go
L='now,k3,k3:2=1'
for pad in (0,3):
  for n in (.5,1,2,4,8,25.5,60):
    if pad and n<8: continue
    go([mk('step',N,t,n,sparse=1,one_in=o) for t in (.5,.3) for N in (2,5,8,9,16) for o in (256,16)],L,3,BLOCK=.02,SETS=3 if n<30 else 2,PAD=pad)
go([mk('step',N,t,n,sparse=1,one_in=64) for t in (.5,.3) for N in (17,24,32,48,64) for n in (.5,1,2)],L,3,BLOCK=.02,SETS=3)
