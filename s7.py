import sys; sys.path.insert(0,'/root/repo/_work/exp')
from sw import mk,go
L='now,'+','.join('k3:4=%d'%x for x in (0,20480,24576,32768,40960,53248))
go([mk('server',N,t,n) for n in (16.7,8,40) for N in (17,24,32) for t in (.5,.3)],L,3,BLOCK=.02,SETS=3)
L='now,k3,k3:7=17,k3:7=19,k3:7=2'
go([mk('worker',8,.5,n,sparse=s,one_in=256) for n in (.3,1,2,4,6,9.4,16,30) for s in (0,1)],L,3,BLOCK=.02,SETS=4)
